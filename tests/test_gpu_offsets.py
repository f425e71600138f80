"""Device offsets that are not the ones the host copies hold (a stale copy):
every buffer is sized from the host's, so whatever the device's say, nothing is
written outside the buffers, and a schedule of more work than the host counted
is reported."""
import numpy as np
import pytest

from paper_2511_06077_amd import workload as W
from test_gpu_guards import Guarded

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def offsets(counts):
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)


EVEN, ONE_LONG = [2048] * 8, [16384 - 7] + [1] * 7


# target groups that the host did not count; more units than the host counted;
# offsets that do not ascend (refused by the scheduler)
@pytest.mark.parametrize("d,h", [(256, 8), (128, 4)])
@pytest.mark.parametrize("L,m,dev_L,dev_m,status", [
    (EVEN, [1] * 8, EVEN, [2, 0] * 4, "ok"),
    (EVEN, [1] * 8, EVEN, [0, 0, 0, 0, 2, 2, 2, 2], "ok"),
    (ONE_LONG, [1] * 8, EVEN, [1] * 8, "invalid"),
    (EVEN, [1] * 8, [4000, -2000, 3000, 1144] + [2560] * 4, [3, -4, 7, 0, 0, 1, 0, 1], "invalid")])
def test_reordered_backward_stays_inside_its_buffers(torch, d, h, L, m, dev_L, dev_m, status):
    from paper_2511_06077_amd import stca
    from paper_2511_06077_amd.device import DeviceBatch, to_device
    M = 128 // h  # targets of a group
    b = W.make_custom_batch("goff", L, [M * x for x in m], d_model=d, n_heads=h, n_layers=2, dtype="bf16", seed=41,
                            with_grad=True)
    db = DeviceBatch(b, backward=True, bwd="reordered", chunk_blocks=8)
    db.hoff.copy_(torch.from_numpy(offsets(dev_L)))
    db.toff.copy_(torch.from_numpy(offsets([M * x for x in dev_m])))
    nt, nh, n, F = b.n_tgt_total, b.n_hist, 2, b.wl.ffn_hidden
    sizes = {"dhist": nh * d, "dtgt": nt * d, "dwq": n * d * d, "dwk": n * d * d, "dwv": n * d * d,
             "dwo": n * d * d, "dw1": n * d * F, "dw2": n * F * d}
    g = {k: Guarded(torch, 4 * v) for k, v in sizes.items()}
    ws = Guarded(torch, db.bws_bytes)
    dw = stca.wgrads(*(g[k].ptr for k in ("dwq", "dwk", "dwv", "dwo", "dw1", "dw2")))
    stca.stca_backward(db.dims, db.batch, db.hist, db.tgt, db.weights, to_device(b.grad_out, "cuda"), g["dhist"].ptr,
                       g["dtgt"].ptr, dw, ws.ptr, db.bws_bytes, db.stream())
    got = stca.stca_device_status(ws.ptr, db.stream())
    assert got == (stca.STCA_OK if status == "ok" else stca.STCA_ERR_INVALID_ARG)
    bad = [k for k, v in {"ws": ws, **g}.items() if not v.intact()]
    assert not bad, bad


# a forward of few targets makes room for as many chunk records as the host's
# lengths have chunks (47 of 3 blocks each here); the device copy shows one
# request twice as long, whose history then goes out in longer chunks
def test_few_target_forward_stays_inside_its_buffers(torch):
    from oracle import stca_oracle as O
    from paper_2511_06077_amd import stca
    from paper_2511_06077_amd.device import DeviceBatch
    kw = dict(d_model=256, n_heads=8, n_layers=2, dtype="bf16", seed=43)
    b = W.make_custom_batch("foff", [4512, 4480], [40, 40], **kw)
    dev = W.make_custom_batch("foff", [8960, 32], [40, 40], **kw)  # the device's offsets
    db = DeviceBatch(b)
    full = DeviceBatch(dev)
    db.hist.copy_(full.hist)
    db.tgt.copy_(full.tgt)
    db.hoff.copy_(full.hoff)
    ws, out = Guarded(torch, db.ws_bytes), Guarded(torch, 2 * b.n_tgt_total * 256)
    stca.stca_forward(db.dims, db.batch, db.hist, db.tgt, full.weights, out.ptr, None, ws.ptr, db.ws_bytes,
                      db.stream())
    assert stca.stca_device_status(ws.ptr, db.stream()) == stca.STCA_OK
    assert ws.intact() and out.intact()
    y = out.view(torch, torch.bfloat16, (b.n_tgt_total, 256)).float().cpu().numpy()
    ref = O.forward(dev.f64())["out"]
    assert float((np.abs(y - ref).max(1) / np.abs(ref).max(1)).max()) <= 2e-2
