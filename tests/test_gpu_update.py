"""GPU: the target update at the edges of its cut (groups of 4, 8, 16 and 32
targets, hidden layer over 1, 2 or 4 workgroups) against the oracle."""
import numpy as np
import pytest

from oracle import stca_oracle as O
from paper_2511_06077_amd import workload as W

pytestmark = pytest.mark.gpu


def rowerr(y, ref):
    return float((np.abs(y - ref).max(-1) / np.maximum(np.abs(ref).max(-1), 1e-30)).max())


# totals around the group and split limits, given at 256 CUs and scaled to the
# card's: 4 targets x 4 splits up to 256, 8 x 4 up to 512, 16 x 4 up to 1024,
# 16 x 2 up to 2048, 16 x 1 up to 4096, then 32
@pytest.mark.parametrize("nt", [1, 5, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
def test_update_cut(nt):
    import torch
    from paper_2511_06077_amd.device import DeviceBatch
    nt = nt // 256 * torch.cuda.get_device_properties(0).multi_processor_count + nt % 256
    m = []
    while sum(m) < nt:
        m.append(min(61, nt - sum(m)))
    L = [5 + 37 * (r % 3) for r in range(len(m))]
    b = W.make_custom_batch("update", L, m, d_model=256, n_heads=8, n_layers=2, dtype="bf16", seed=31)
    db = DeviceBatch(b, keep_saved=True)
    y = db.forward().float().cpu().numpy()
    again = db.forward()
    torch.cuda.synchronize()
    assert np.array_equal(again.float().cpu().numpy(), y)
    ref = O.forward(b.f64())
    # the bar of the bf16 forward (tests/test_gpu_forward.py): 2e-2 per row
    assert rowerr(y, ref["out"]) <= 2e-2
    for i in range(2):
        assert rowerr(db.saved_tensor("a")[i].cpu().numpy(), ref["a"][i]) <= 2e-2
