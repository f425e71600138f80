"""GPU: the device scheduler at the edges of its two ways to share the units
(up to 1024 requests a thread each, then runs of requests), through the
forward against the oracle."""
import numpy as np
import pytest

from oracle import stca_oracle as O
from paper_2511_06077_amd import workload as W

pytestmark = pytest.mark.gpu


def rowerr(y, ref):
    return float((np.abs(y - ref).max(-1) / np.maximum(np.abs(ref).max(-1), 1e-30)).max())


@pytest.mark.parametrize("requests,m_hi,host", [(1, 70, True), (1023, 3, True), (1024, 40, False), (1025, 40, False),
                                                (1500, 70, True), (300, 130, True)])
def test_schedule(requests, m_hi, host):
    """Empty target segments, both width classes (33.. targets, the narrow last
    group of a wide request), chunks, device and host offsets."""
    import torch
    from paper_2511_06077_amd.device import DeviceBatch
    rng = np.random.default_rng(requests)
    m = np.where(rng.random(requests) < 0.9, rng.integers(0, 4, requests), rng.integers(0, m_hi + 1, requests))
    m[0] = m_hi
    L = rng.integers(1, 40, requests)
    L[-1] = 700
    b = W.make_custom_batch("sched", L, m, d_model=64, n_heads=2, n_layers=1, dtype="bf16", seed=41)
    ref = O.forward(b.f64())["out"]
    for chunk in (0, 1):
        db = DeviceBatch(b, host_offsets=host, chunk_blocks=chunk)
        y = db.forward().float().cpu().numpy()
        assert db.device_status() == 0
        assert rowerr(y, ref) <= 2e-2  # the bar of the bf16 forward


@pytest.mark.parametrize("d,h", [(256, 8), (128, 4)])
@pytest.mark.parametrize("L,m,host", [([9001], [40], True), ([9001], [40], False), ([4100], [3], True),
                                      ([5000, 70, 1, 900, 2048], [3, 64, 2, 33, 12], True),
                                      ([700, 2000, 64, 33], [1, 2, 40, 64], True)])
def test_few_requests(L, m, host, d, h):
    """Few requests: more than 16 history chunks each, and batches that mix both
    widths and the reordered form in one attention launch."""
    import torch
    from paper_2511_06077_amd.device import DeviceBatch
    b = W.make_custom_batch("few", L, m, d_model=d, n_heads=h, n_layers=2, dtype="bf16", seed=43)
    db = DeviceBatch(b, host_offsets=host, keep_saved=True)
    y = db.forward().float().cpu().numpy()
    again = db.forward()
    torch.cuda.synchronize()
    assert np.array_equal(again.float().cpu().numpy(), y) and db.device_status() == 0
    ref = O.forward(b.f64())
    assert rowerr(y, ref["out"]) <= 2e-2
    for i in range(2):
        assert rowerr(db.saved_tensor("a")[i].cpu().numpy(), ref["a"][i]) <= 2e-2


def test_profiled_labels_of_shared_launches():
    """The places of kernels whose work runs inside another launch are labelled
    "none": the schedules and the packing, and of a batch of three forms (one,
    32 and 64 targets a request) the attention's."""
    import torch
    from paper_2511_06077_amd import stca
    from paper_2511_06077_amd.device import DeviceBatch
    b = W.make_custom_batch("labels", [300, 200, 400], [1, 32, 64], d_model=256, n_heads=8, n_layers=2, dtype="bf16",
                            seed=47)
    db = DeviceBatch(b)
    n = stca.stca_forward_launch_count(db.dims, db.batch)
    ev = stca.HipEvents(n + 1)
    try:
        stca.stca_forward_profiled(db.dims, db.batch, db.hist, db.tgt, db.weights, db.out, None, db.ws, db.ws_bytes,
                                   db.stream(), ev.ev, ev.labels)
        torch.cuda.synchronize()
        labels = [ev.label(k) for k in range(n)]
    finally:
        ev.close()
    assert labels == ["setup", "none", "none", "update"] + 2 * ["reord_u", "attn_mixed", "none", "none",
                                                                "reord_merge", "update"]
