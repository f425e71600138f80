"""GPU parity of the backward with the exact fp32 attention at its edges: target
batches of 16, passes of 64 targets (later passes add to the rows the first
wrote), history tails and chunks; on bf16 storage it follows the precise
recomputation for requests of more than 32 targets."""
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


# one target over and under a batch (16) and a pass (64), three passes
@pytest.mark.parametrize("d,h,dtype", [(256, 8, "bf16"), (128, 4, "bf16"), (64, 2, "bf16"), (128, 2, "bf16"),
                                       (64, 4, "f32"), (64, 2, "f32"), (128, 2, "f32")])
def test_many_targets(torch, d, h, dtype):
    # the first seed whose ReLU inputs all lie further than 2e-6 from zero: fp32
    # states differ from the oracle's by up to about 1e-6, and a gate within
    # that falls either way in any evaluation (at 2.4e-7 both this form and
    # the generic one flip it, 2.5e-2 of dw1's maximum in so small a batch)
    for seed in range(107, 127):
        b = W.make_custom_batch("gmany", [1, 33, 130, 64, 7, 500, 45], [33, 64, 0, 65, 129, 17, 16], d_model=d,
                                n_heads=h, n_layers=2, dtype=dtype, seed=seed, with_grad=True)
        if np.abs(O.forward(b.f64())["pre"]).min() > 2e-6:
            break
    else:
        pytest.fail("no seed without a gate near zero")
    for kw in ({}, {"chunk_blocks": 3}):
        g = gpu_grads(torch, b, **kw)
        check(b, g, TOL[dtype])
        assert not np.any(g["dhist"][b.hist_off[2]:b.hist_off[3]])
