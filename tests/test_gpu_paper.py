"""GPU parity of the paper-exact stack (stca_forward_paper through the C ABI)
against the fp64 paper oracle on the same seeded inputs.

Compared: the head token z, and per layer the transformed history X~^(i), the
query q^(i), the head concatenation a^(i), the layer summary o^(i) and the
log-sum-exp.  Metric and bars as for the configuration-mode forward (per-row
max-norm error; 1e-4 with fp32 storage, 2e-2 with bf16 storage).
"""
import numpy as np
import pytest

from oracle import stca_paper_oracle as P
from paper_2511_06077_amd import workload as W
from test_gpu_forward import LSE_ABS, LSE_REL, TOL, rowerr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def run_paper(torch, b, weights, keep_saved=True, host_offsets=True, chunk_blocks=0):
    from paper_2511_06077_amd.device import PaperDeviceBatch
    db = PaperDeviceBatch(b, weights, keep_saved=keep_saved, host_offsets=host_offsets, chunk_blocks=chunk_blocks)
    z = db.forward()
    torch.cuda.synchronize()
    out = {"z": z.float().cpu().numpy().astype(np.float64)}
    if keep_saved:
        for k in ("q", "a", "o", "lse", "xt"):
            out[k] = db.saved_tensor(k).cpu().numpy().astype(np.float64)
    return out, db


def check(b, weights, got, tol, tgt_rows=None, hist_rows=None, requests=None):
    """Compare against the oracle; with `requests`, the oracle runs on those
    requests alone (their rows tgt_rows / hist_rows of the GPU batch)."""
    if requests is None:
        ref = P.forward_paper(W.paper_f64(b, weights))
        tgt_rows = slice(None)
        hist_rows = slice(None)
    else:
        sub = W.make_batch(b.wl, requests=requests)
        ref = P.forward_paper(W.paper_f64(sub, weights))
    M = b.wl.n_layers
    e = {"z": rowerr(got["z"][tgt_rows], ref["z"])}
    if "a" in got:
        e["a"] = max(rowerr(got["a"][i][tgt_rows], ref["a"][i]) for i in range(M))
        e["q"] = max(rowerr(got["q"][i][tgt_rows], ref["q"][i]) for i in range(M))
        e["o"] = max(rowerr(got["o"][tgt_rows, i], ref["o"][i]) for i in range(M))
        e["xt"] = max(rowerr(got["xt"][i][hist_rows], ref["xt"][i]) for i in range(M))
        e["lse"] = float(np.abs(got["lse"][:, tgt_rows] - ref["lse"]).max()) if ref["lse"].size else 0.0
    dt = "f32" if tol < 1e-3 else "bf16"
    lse_bar = max(LSE_ABS[dt], LSE_REL[dt] * float(np.abs(ref["lse"]).max())) if ref["lse"].size else 0.0
    print(f"[paper parity] {b.wl.name}: " + " ".join(f"err({k})={v:.2e}" for k, v in e.items())
          + f" (lse bar {lse_bar:.1e})", flush=True)
    for k, v in e.items():
        assert v <= (lse_bar if k == "lse" else tol), (k, v)


EDGE_L = [1, 7, 31, 32, 33, 63, 65, 200, 1023, 1, 40, 64, 129]
EDGE_M = [1, 17, 0, 64, 33, 32, 1, 15, 2, 0, 31, 16, 70]


@pytest.mark.parametrize("dtype,d,h,n,F", [("bf16", 256, 8, 2, 1024), ("bf16", 128, 4, 3, 512),
                                           ("bf16", 64, 2, 1, 256), ("f32", 64, 2, 2, 256),
                                           ("f32", 32, 2, 3, 64)])
@pytest.mark.parametrize("chunk", [0, 1])
def test_paper_edge_parity(torch, dtype, d, h, n, F, chunk):
    """Ragged tails (history lengths not multiples of 32, 0..70 targets per
    request, empty target segments) on both kernel families."""
    b = W.make_custom_batch("paper_edge", EDGE_L, EDGE_M, d_model=d, n_heads=h, n_layers=n, dtype=dtype, seed=61)
    b.wl = W.Workload(b.wl.name, b.wl.n_requests, d, h, n, dtype, b.wl.seed, ffn_mult=F // d)
    weights = W.make_paper_weights(b.wl)
    got, db = run_paper(torch, b, weights, chunk_blocks=chunk)
    from paper_2511_06077_amd import stca
    assert stca.stca_path(db.dims) == (1 if dtype == "bf16" else 0)
    check(b, weights, got, TOL[dtype])


def test_paper_device_offsets(torch):
    """Without host offsets (device scheduler only) the result is the same."""
    b = W.make_custom_batch("paper_dev", [300, 64, 1000], [5, 40, 1], d_model=256, n_heads=8, n_layers=2,
                            dtype="bf16", seed=62)
    weights = W.make_paper_weights(b.wl)
    got, _ = run_paper(torch, b, weights, keep_saved=False, host_offsets=False)
    got2, _ = run_paper(torch, b, weights, keep_saved=False, host_offsets=True)
    # the same chunks (of 8 blocks) and the same order of every sum either way
    assert np.array_equal(got["z"], got2["z"])
    check(b, weights, got, TOL["bf16"])


def test_paper_headline_shape_sampled(torch):
    """128 requests x 32 targets, L = 10240, d = 256, 8 heads, 4 layers, r = 4
    (bf16), in the benchmark's launch configuration; the oracle checks a
    seeded sample of 16 requests (requests are independent), on every saved
    tensor including the transformed histories."""
    from paper_2511_06077_amd.device import PaperDeviceBatch
    wl = W.WORKLOADS[W.HEADLINE]
    b = W.make_batch(wl)
    weights = W.make_paper_weights(wl)
    db = PaperDeviceBatch(b, weights, keep_saved=True)
    z = db.forward()
    torch.cuda.synchronize()
    req = np.sort(np.random.default_rng(6).choice(wl.n_requests, 16, replace=False))
    trow = torch.from_numpy(np.concatenate([np.arange(b.tgt_off[r], b.tgt_off[r + 1]) for r in req])).cuda()
    hrow = torch.from_numpy(np.concatenate([np.arange(b.hist_off[r], b.hist_off[r + 1]) for r in req])).cuda()
    np64 = lambda x: x.float().cpu().numpy().astype(np.float64)  # noqa: E731
    got = {"z": np64(z[trow]), "q": np64(db.saved_tensor("q")[:, trow]), "a": np64(db.saved_tensor("a")[:, trow]),
           "o": np64(db.saved_tensor("o")[trow]), "lse": np64(db.saved_tensor("lse")[:, trow]),
           "xt": np64(db.saved_tensor("xt")[:, hrow])}
    check(b, weights, got, TOL["bf16"], tgt_rows=slice(None), hist_rows=slice(None), requests=req)


def test_paper_profiled_labels(torch):
    from paper_2511_06077_amd import stca
    b = W.make_custom_batch("paper_prof", [100, 37], [3, 9], d_model=128, n_heads=4, n_layers=3, dtype="bf16",
                            seed=63)
    weights = W.make_paper_weights(b.wl)
    from paper_2511_06077_amd.device import PaperDeviceBatch
    db = PaperDeviceBatch(b, weights)
    n = stca.stca_paper_launch_count(db.dims, db.batch)
    ev = stca.HipEvents(n + 1)
    try:
        stca.stca_forward_paper_profiled(db.dims, db.batch, db.hist, db.tgt, db.weights, db.z, None, db.ws,
                                         db.ws_bytes, db.stream(), ev.ev, ev.labels)
        torch.cuda.synchronize()
        labels = [ev.label(k) for k in range(n)]
        assert labels.count("swiglu_ln") == 3 and "?" not in labels
        assert all(ev.elapsed_ms(0, k + 1) >= 0 for k in range(n))
        z1 = db.z.float().cpu().numpy()
        db.forward()
        torch.cuda.synchronize()
        assert np.array_equal(z1, db.z.float().cpu().numpy())
    finally:
        ev.close()


# F = 2 d and 3 d: the target stage without a compile-time chunk count, its
# hidden columns over two workgroups (2 chunks) and one (3 chunks)
@pytest.mark.parametrize("d,h,mult", [(256, 8, 2), (256, 8, 3), (128, 4, 2), (128, 4, 6), (64, 2, 8)])
def test_paper_other_ffn_width(torch, d, h, mult):
    b = W.make_custom_batch("paper_ffn", EDGE_L, EDGE_M, d_model=d, n_heads=h, n_layers=2, dtype="bf16", seed=64)
    b.wl = W.Workload(b.wl.name, b.wl.n_requests, d, h, 2, "bf16", b.wl.seed, ffn_mult=mult)
    weights = W.make_paper_weights(b.wl)
    got, _ = run_paper(torch, b, weights)
    check(b, weights, got, TOL["bf16"])


# more target groups of 32 than half of the CUs take one workgroup each (few
# rows a request; the last group partial), exactly half two
@pytest.mark.parametrize("extra", [0, 5])
def test_paper_target_splits(torch, extra):
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    m = [32] * (cu // 2) + ([extra] if extra else [])
    b = W.make_custom_batch("paper_split", [3 + r % 5 for r in range(len(m))], m, d_model=256, n_heads=8, n_layers=2,
                            dtype="bf16", seed=65)
    weights = W.make_paper_weights(b.wl)
    got, _ = run_paper(torch, b, weights, keep_saved=False)
    check(b, weights, got, TOL["bf16"])


# the history transform's four-wave workgroups up to 128 rows a CU, eight-wave ones
# beyond (the last of 256 rows holds one)
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_paper_history_rows(torch, extra):
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    rows = 128 * cu + extra
    b = W.make_custom_batch("paper_rows", [rows // 2, rows - rows // 2], [3, 2], d_model=64, n_heads=2, n_layers=1,
                            dtype="bf16", seed=66)
    weights = W.make_paper_weights(b.wl)
    got, _ = run_paper(torch, b, weights)
    check(b, weights, got, TOL["bf16"])
