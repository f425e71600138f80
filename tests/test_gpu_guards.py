"""Every buffer the library writes (out, saved, workspace, the gradients and
the training record) is bracketed by guard regions filled with a known byte
pattern; after the forward and the backward on the ragged edge batch the
guards must be untouched, and the results must be the same as through
ordinary buffers."""
import numpy as np
import pytest

from paper_2511_06077_amd import workload as W

pytestmark = pytest.mark.gpu

GUARD = 64 * 1024  # bytes on each side (a multiple of 256: keeps alignment)
PATTERN = 0xA5


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


class Guarded:
    """A device buffer of `nbytes` with GUARD pattern bytes before and after."""

    def __init__(self, torch, nbytes):
        self.n = int(nbytes)
        self.raw = torch.full((self.n + 2 * GUARD,), PATTERN, dtype=torch.uint8, device="cuda")
        self.ptr = self.raw.data_ptr() + GUARD

    def view(self, torch, dtype, shape):
        return self.raw[GUARD:GUARD + self.n].view(dtype).view(*shape)

    def intact(self):
        head = self.raw[:GUARD]
        tail = self.raw[GUARD + self.n:]
        return bool((head == PATTERN).all().item()) and bool((tail == PATTERN).all().item())


EDGE_L = [1, 7, 31, 32, 33, 63, 65, 200, 1023, 1, 40, 64]
EDGE_M = [1, 17, 0, 64, 33, 32, 1, 15, 2, 0, 31, 16]
NARROW_M = [1, 17, 0, 32, 31, 32, 1, 15, 2, 0, 31, 16]  # at most 32 targets: the fused backward


@pytest.mark.parametrize("dtype,d,h,m,forms", [
    ("bf16", 256, 8, EDGE_M, {}), ("bf16", 256, 8, EDGE_M, {"kv": "materialize"}),
    ("bf16", 256, 8, [i % 5 for i in range(12)], {"attn": "reordered"}),
    ("bf16", 128, 4, NARROW_M, {}), ("f32", 64, 2, EDGE_M, {})])
def test_forward_and_backward_stay_inside_their_buffers(torch, dtype, d, h, m, forms):
    from paper_2511_06077_amd import stca
    from paper_2511_06077_amd.device import DeviceBatch, to_device
    b = W.make_custom_batch("guard", EDGE_L, m, d_model=d, n_heads=h, n_layers=2, dtype=dtype, seed=23,
                            with_grad=True)
    db = DeviceBatch(b, keep_saved=True, backward=True, **forms)  # the reference run, ordinary buffers
    y_ref = db.forward().clone()
    saved_ref = db.saved.clone()
    dout = to_device(b.grad_out, "cuda")
    g_ref = db.backward(dout)
    torch.cuda.synchronize()

    es = 2 if dtype == "bf16" else 4
    nt, nh, n, F = b.n_tgt_total, b.n_hist, 2, b.wl.ffn_hidden
    out = Guarded(torch, nt * d * es)
    saved = Guarded(torch, db.saved_bytes)
    ws = Guarded(torch, db.ws_bytes)
    stca.stca_forward(db.dims, db.batch, db.hist, db.tgt, db.weights, out.ptr, saved.ptr, ws.ptr, db.ws_bytes,
                      db.stream())
    sizes = {"dhist": nh * d, "dtgt": nt * d, "dwq": n * d * d, "dwk": n * d * d, "dwv": n * d * d,
             "dwo": n * d * d, "dw1": n * d * F, "dw2": n * F * d}
    gb = {k: Guarded(torch, 4 * v) for k, v in sizes.items()}
    bws = Guarded(torch, db.bws_bytes)
    dw = stca.wgrads(*(gb[k].ptr for k in ("dwq", "dwk", "dwv", "dwo", "dw1", "dw2")))
    stca.stca_backward(db.dims, db.batch, db.hist, db.tgt, db.weights, dout, gb["dhist"].ptr, gb["dtgt"].ptr, dw,
                       bws.ptr, db.bws_bytes, db.stream())
    rec = None
    if db.record is not None:
        # the two-call training step: record and gradients through guarded buffers too
        rec = Guarded(torch, db.record.numel())
        out2 = Guarded(torch, nt * d * es)
        bws2 = Guarded(torch, db.bws_bytes)
        stca.stca_forward_train(db.dims, db.batch, db.hist, db.tgt, db.weights, out2.ptr, rec.ptr, bws2.ptr,
                                db.bws_bytes, db.stream())
        gb2 = {k: Guarded(torch, 4 * v) for k, v in sizes.items()}
        dw2 = stca.wgrads(*(gb2[k].ptr for k in ("dwq", "dwk", "dwv", "dwo", "dw1", "dw2")))
        stca.stca_backward_record(db.dims, db.batch, db.hist, db.tgt, db.weights, rec.ptr, dout, gb2["dhist"].ptr,
                                  gb2["dtgt"].ptr, dw2, bws2.ptr, db.bws_bytes, db.stream())
    torch.cuda.synchronize()

    bufs = {"out": out, "saved": saved, "ws": ws, "bws": bws, **{"g_" + k: v for k, v in gb.items()}}
    if rec is not None:
        bufs.update({"record": rec, "out2": out2, "bws2": bws2, **{"g2_" + k: v for k, v in gb2.items()}})
    bad = [k for k, v in bufs.items() if not v.intact()]
    print(f"[guard] {dtype} d={d} forms={forms}: {len(bufs)} buffers checked, overwritten guards: {bad}", flush=True)
    assert not bad, bad
    # the same results as through the ordinary buffers
    sdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    assert torch.equal(out.view(torch, sdt, (nt, d)), y_ref)
    lay = db.layout
    for name, cols in (("s", d), ("a", d), ("u", d), ("lse", h)):
        off, cnt = getattr(lay, name), 4 * n * nt * cols
        assert torch.equal(saved.raw[GUARD + off:GUARD + off + cnt], saved_ref[off:off + cnt]), name
    # (every sum has a fixed order)
    for k, v in sizes.items():
        assert torch.equal(gb[k].view(torch, torch.float32, (v,)), g_ref[k].reshape(-1)), k
