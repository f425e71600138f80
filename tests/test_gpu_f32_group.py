"""GPU parity of the fp32-storage path's grouped products where a product's
tiling changes: output tiles of 64 with remainders, 32-deep k tiles with
remainders, long reductions split over K from 1024 rows on (several splits with
a short last one), requests without targets."""
import numpy as np
import pytest

from oracle import stca_oracle as O
from paper_2511_06077_amd import workload as W
from test_gpu_backward import TOL, check, gpu_grads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


# d x d weight gradients over 2, 63, 65 and 1023 rows in one piece, over 1024,
# 1100 and 2113 split (2113 = 14 chunks of 160, the last of 33); up to
# 130 targets.  (Not over one row: its softmax weight is 1 and dW_Q, dW_K are zero
# in the oracle, so a relative bound is none; the GPU leaves dP - D, which its
# roundings bound by about 2^-23 |dP|.)
@pytest.mark.parametrize("d,h,L,m", [(64, 2, [2], [1]), (64, 2, [60, 3], [1, 0]), (128, 2, [33, 32], [64, 1]),
                                     (64, 8, [1000, 23], [3, 5]), (64, 2, [1024], [4]), (128, 4, [1100], [65]),
                                     (64, 1, [2048, 65], [129, 1])])
def test_f32_products(torch, d, h, L, m):
    from paper_2511_06077_amd.device import DeviceBatch
    b = W.make_custom_batch("gf32", L, m, d_model=d, n_heads=h, n_layers=2, dtype="f32", seed=97, with_grad=True)
    y = DeviceBatch(b).forward().cpu().numpy().astype(np.float64)
    ref = O.forward(b.f64())["out"]
    # (sums of at most 4 d = 512 fp32 terms through two layers: 2^-24 sqrt(512) = 1.3e-6 a product)
    assert np.abs(y - ref).max() <= 2e-5 * np.abs(ref).max()
    check(b, gpu_grads(torch, b), TOL["f32"])


# the same call gives the same bits: the parts of a split product are summed in
# one order (rows 1024, 1100 and 2113 split the weight gradients over K, as
# 1100 targets do, and d = 1024 the forward's products)
@pytest.mark.parametrize("d,h,L,m", [(64, 2, [1024], [4]), (128, 4, [1100], [65]), (64, 1, [2048, 65], [129, 1]),
                                     (64, 2, [40, 50], [600, 500]), (1024, 16, [70, 30], [3, 2])])
def test_f32_repeats(torch, d, h, L, m):
    from paper_2511_06077_amd.device import DeviceBatch, to_device
    b = W.make_custom_batch("gf32r", L, m, d_model=d, n_heads=h, n_layers=2, dtype="f32", seed=97, with_grad=True)
    db = DeviceBatch(b, backward=True)
    dout = to_device(b.grad_out, "cuda")
    y, g = db.forward().clone(), db.backward(dout)
    ref = O.forward(b.f64())["out"]
    # (sums of at most 4 d fp32 terms through two layers: 2^-24 sqrt(4096) = 4e-6 a product)
    assert np.abs(y.cpu().numpy() - ref).max() <= 4e-5 * np.abs(ref).max()
    for _ in range(3):
        y2, g2 = db.forward(), db.backward(dout)
        assert torch.equal(y, y2)
        for k in g:
            assert torch.equal(g[k], g2[k]), k


# dhist adds dK W_K^T and dV W_V^T of each layer as two sums of d terms.  Mean
# error over eight input sets: 5.6e-7 and 7.3e-7 of the norm; in one accumulator
# of 2 d terms 5.8e-7 and 7.6e-7.
@pytest.mark.parametrize("d,h,L,m,bar", [(64, 2, [256] * 4, [4] * 4, 5.7e-7), (128, 4, [300, 500], [3, 7], 7.4e-7)])
def test_f32_dhist_error(torch, d, h, L, m, bar):
    errs = []
    for seed in range(1, 9):
        b = W.make_custom_batch("x", L, m, d_model=d, n_heads=h, n_layers=2, dtype="f32", seed=seed, with_grad=True)
        f = b.f64()
        ref = O.backward(f, f["grad_out"])["dhist"]
        errs.append(np.linalg.norm(gpu_grads(torch, b)["dhist"] - ref) / np.linalg.norm(ref))
    print(f"[grad] dhist error {np.mean(errs):.2e}", flush=True)
    assert np.mean(errs) <= bar


# 2^24 workgroups and more in one group of products (K and V of 2^29 rows, d = 8):
# rows from the ends and the middle of the batch against the oracle
def test_f32_many_tiles(torch):
    from paper_2511_06077_amd.device import DeviceBatch
    R, per = 4096, 1 << 17
    m = np.zeros(R, dtype=np.int64)
    used = [0, R // 2 + 1, R - 1]
    m[used] = 2
    small = W.make_custom_batch("gtiles", [per] * len(used), [2] * len(used), d_model=8, n_heads=1, n_layers=1,
                                dtype="f32", seed=5)
    hist = torch.zeros((R * per, 8), device="cuda")
    src = torch.from_numpy(small.hist).cuda()
    for i, r in enumerate(used):
        hist[r * per:(r + 1) * per] = src[i * per:(i + 1) * per]
    wl = W.Workload("gtiles", R, 8, 1, 1, "f32", seed=5, ffn_mult=4)
    b = W.Batch(wl, np.arange(R), np.full(R, per), m, (np.arange(R + 1) * per).astype(np.int32),
                np.concatenate([[0], np.cumsum(m)]).astype(np.int32), None, None, small.weights)
    db = DeviceBatch.from_tensors(b, hist, torch.from_numpy(small.tgt).cuda(),
                                  {k: torch.from_numpy(v).cuda() for k, v in small.weights.items()})
    y = db.forward().cpu().numpy()
    ref = O.forward(small.f64())["out"]
    # (softmax sums of 131072 fp32 terms in runs of at most 8192)
    assert np.abs(y - ref).max() <= 2e-5 * np.abs(ref).max()
