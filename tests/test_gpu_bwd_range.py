"""GPU: the backward over the range that bf16 histories may use.  Scaling column
c of the history by 2^e_c and row c of W_K and W_V by 2^-e_c is exact in bf16 and
leaves K, V and every gradient but dhist, dW_K and dW_V (scaled in turn) as they
are, so each form is held to the oracle's gradients of the unscaled batch, at the
bar of test_gpu_backward."""
import dataclasses

import numpy as np
import pytest

from paper_2511_06077_amd import workload as W
from test_gpu_backward import TOL, check, gpu_grads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def exponents(kind, d):
    e = np.zeros(d, dtype=np.int64)
    if kind == "large":  # |x| up to 4e6, fp16's largest is 65504
        e[:] = 20
    elif kind == "small":  # |x| about 6e-8, fp16's smallest step; |q W_K^T| about 2e7
        e[:] = -24
    elif kind == "mixed":
        e[1::2], e[::2] = 18, -8
    elif kind == "one_block":  # two rows with one large entry
        e[0] = 20
    return e


def scaled(b, e):
    """(b with its columns and rows scaled, the gradients' scaling back)"""
    def times(bits, f):
        return W.to_bf16_bits((W.bf16_bits_to_f32(bits).astype(np.float64) * f).astype(np.float32))
    f = 2.0 ** e
    w = {**b.weights, **{k: times(b.weights[k], (1 / f)[:, None]) for k in ("wk", "wv")}}
    s = dataclasses.replace(b, hist=times(b.hist, f), weights=w)
    return s, {"dhist": f, "dwk": (1 / f)[:, None], "dwv": (1 / f)[:, None]}


@pytest.mark.parametrize("d,h", [(256, 8), (128, 4)])
@pytest.mark.parametrize("form", ["reordered", "fused"])
@pytest.mark.parametrize("kind", ["large", "small", "mixed", "one_block"])
def test_history_range(torch, kind, form, d, h):
    # (seed 74: every ReLU input lies further than 1e-5 from zero in all of these;
    # the recomputed states are off by about 1e-6, and a gate within that falls
    # either way, which alone moves a column of dW_1 by some 3e-2 in so small a batch)
    mmax = 128 // h
    b = W.make_custom_batch("grange", [1, 33, 130, 64, 7, 700, 45], [2, mmax, 0, mmax - 1, 1, 5, 3], d_model=d,
                            n_heads=h, n_layers=2, dtype="bf16", seed=74, with_grad=True)
    if kind == "one_block":
        b.hist[:, 0] = 0
        b.hist[[100, 301], 0] = W.to_bf16_bits(np.array([3.0, -2.5], dtype=np.float32))
    s, back = scaled(b, exponents(kind, d))
    g = gpu_grads(torch, s, bwd=form, chunk_blocks=4)
    check(b, {k: v * back.get(k, 1.0) for k, v in g.items()}, TOL["bf16"])


def test_history_range_target_groups(torch):
    """The automatic choice's reordered form with two target groups a request."""
    from paper_2511_06077_amd import stca
    from paper_2511_06077_amd.device import DeviceBatch
    rng = np.random.default_rng(6)
    b = W.make_custom_batch("grangegrp", rng.integers(700, 2400, 128), np.where(rng.random(128) < 0.2, 20, 9),
                            d_model=256, n_heads=8, n_layers=2, dtype="bf16", seed=101, with_grad=True)
    s, back = scaled(b, exponents("mixed", 256))
    db = DeviceBatch(s, backward=True)
    assert stca.stca_backward_launch_count(db.dims, db.batch) == 6 + 6 * b.wl.n_layers
    check(b, {k: v * back.get(k, 1.0) for k, v in gpu_grads(torch, s).items()}, TOL["bf16"])


# With W_K, W_V times a power of two and W_Q, W_O divided by it, K is about 1e6
# (past fp16) and V about 6e-8 (fp16's smallest step): with more than 32 targets a
# request the attention is fp32 both ways and every gradient is as without
@pytest.mark.parametrize("d,h", [(256, 8), (128, 4), (64, 2)])
def test_projection_range_many_targets(torch, d, h):
    from oracle import stca_oracle as O
    for seed in range(107, 147):
        b = W.make_custom_batch("gproj", [1, 33, 130, 64, 7, 500, 45], [33, 64, 0, 65, 129, 17, 16], d_model=d,
                                n_heads=h, n_layers=2, dtype="bf16", seed=seed, with_grad=True)
        if np.abs(O.forward(b.f64())["pre"]).min() > 2e-6:  # (as above)
            break
    else:
        pytest.fail("every seed has a gate near zero")
    f = {"wk": 2.0 ** 20, "wq": 2.0 ** -20, "wv": 2.0 ** -24, "wo": 2.0 ** 24}
    w = {k: W.to_bf16_bits(W.bf16_bits_to_f32(v) * np.float32(f.get(k, 1.0))) for k, v in b.weights.items()}
    g = gpu_grads(torch, dataclasses.replace(b, weights=w))
    check(b, {k: v * f.get(k[1:], 1.0) for k, v in g.items()}, TOL["bf16"])
