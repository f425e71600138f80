"""The work that a user of this library has it do, as cases to be timed.

Every case is one call sequence through the public entry points on a packed
ragged batch: a forward of the standard stack (scoring), a training step
(forward and backward) or a forward of the paper-exact stack.  A case is a
dict of plain values:

  kind      "score", "train" or "paper"
  dtype     "bf16" or "f32" (storage of history, targets, weights, output)
  d, heads, layers          model (FFN width 4 d)
  requests, L, m            requests, (lowest, highest) history length and
                            target count as "lo-hi"; drawn uniform, inclusive
  sl        stochastic-length histories (Beta curriculum): L holds the mean
            and the longest length instead
  shape     seed of the lengths and target counts, which belong to the case;
            the seed given to prepare() draws the values

Embeddings are N(0, 1) and weights are scaled by their fan-in, as in
paper_2511_06077_amd/workload.py.
"""
import math

import numpy as np
import torch

from paper_2511_06077_amd import stca
from paper_2511_06077_amd.device import DeviceBatch
from paper_2511_06077_amd.workload import Batch, Workload

FFN_MULT = 4
SL_ALPHA, SL_MIN = 0.02, 8
LN_EPS = 1e-5


def _case(name, kind, requests, L, m, *, dtype="bf16", d=256, heads=8, layers=4, sl=False, shape=0):
    return {"name": name, "kind": kind, "dtype": dtype, "d": d, "heads": heads, "layers": layers,
            "requests": requests, "L": L, "m": m, "sl": sl, "shape": shape}


def listed():
    return [
        # one user's page of candidates, scored as it arrives: what counts is
        # the latency of a single request with a long, odd history
        _case("score_one_request", "score", 1, "9001-9001", "40-40"),
        # a few requests gathered for some milliseconds before scoring
        _case("score_few_requests", "score", 8, "512-10240", "1-64", shape=11),
        # a full serving batch: 10k histories, 32 candidates per request (the
        # benchmark's workload)
        _case("score_full_batch", "score", 128, "10240-10240", "32-32"),
        # a full serving batch as traffic brings it, every length and every
        # number of candidates up to 64
        _case("score_ragged_batch", "score", 256, "512-10240", "1-64", shape=4),
        # one candidate per request (re-scoring, pointwise logging)
        _case("score_one_target", "score", 128, "10240-10240", "1-1"),
        # few users, many candidates each (a late ranking stage)
        _case("score_many_targets", "score", 16, "10240-10240", "256-256"),
        # the smaller model: d = 128, two layers, 1k histories
        _case("score_small_model", "score", 64, "1024-1024", "16-16", d=128, heads=4, layers=2),
        # fp32 storage, forward and backward, at the size of a parity or
        # debugging run
        _case("train_f32", "train", 4, "256-256", "4-4", dtype="f32", d=64, heads=2, layers=2),
        # a training step at the 2k window, 16 targets per request
        _case("train_window", "train", 256, "2048-2048", "16-16"),
        # a training step on a stochastic-length batch: mean 2048, longest 10240
        _case("train_stochastic", "train", 256, "2048-10240", "16-16", sl=True, shape=5),
        # a training step on logged requests with any number of targets up to 64
        _case("train_many_targets", "train", 64, "256-2048", "1-64", shape=7),
        # the paper-exact stack (SwiGLU + LayerNorm history transform) on a
        # ragged serving batch
        _case("paper_ragged_batch", "paper", 64, "512-10240", "1-64", shape=9),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed kinds, sizes over their whole ranges."""
    shape = rng.randrange(1, 1 << 20)
    kind = rng.choice(["score", "score", "score", "score_long", "score_model", "train", "train", "train_f32", "paper"])
    if kind == "score":  # any number of requests, ragged
        hi = _log_int(rng, 300, 10240)
        lo = _log_int(rng, 64, hi)
        R = _log_int(rng, 1, min(256, max(1, 1400000 // hi)))
        mh = _log_int(rng, 1, 64)
        return _case(None, "score", R, f"{lo}-{hi}", f"{rng.randint(1, mh)}-{mh}", shape=shape)
    if kind == "score_long":  # many candidates per request
        hi = _log_int(rng, 1000, 10240)
        lo = _log_int(rng, 500, hi)
        R = _log_int(rng, 1, 16)
        mh = _log_int(rng, 65, 256)
        return _case(None, "score", R, f"{lo}-{hi}", f"{rng.randint(1, mh)}-{mh}", shape=shape)
    if kind == "score_model":  # smaller models
        d = rng.choice([64, 128])
        hi = _log_int(rng, 100, 4096)
        lo = _log_int(rng, 32, hi)
        mh = _log_int(rng, 2, 48)
        return _case(None, "score", _log_int(rng, 1, 128), f"{lo}-{hi}", f"1-{mh}", d=d, heads=d // 32,
                     layers=rng.randint(1, 4), shape=shape)
    if kind == "train":
        if rng.random() < 0.3:
            mean = _log_int(rng, 512, 2048)
            R = _log_int(rng, 16, 256)
            return _case(None, "train", R, f"{mean}-{mean * 5}", f"{rng.randint(1, 16)}-16", sl=True, shape=shape)
        mh = rng.choice([_log_int(rng, 1, 16), rng.randint(8, 32), rng.randint(33, 64)])
        hi = _log_int(rng, 128, 2048)
        lo = _log_int(rng, 64, hi)
        R = _log_int(rng, 2, 256 if mh <= 32 else 64)
        return _case(None, "train", R, f"{lo}-{hi}", f"{rng.randint(1, mh)}-{mh}", shape=shape)
    if kind == "train_f32":
        d = rng.choice([64, 128])
        hi = _log_int(rng, 64, 512)
        lo = _log_int(rng, 16, hi)
        mh = _log_int(rng, 1, 16)
        return _case(None, "train", _log_int(rng, 1, 16), f"{lo}-{hi}", f"1-{mh}", dtype="f32", d=d, heads=d // 32,
                     layers=2, shape=shape)
    hi = _log_int(rng, 300, 10240)
    lo = _log_int(rng, 64, hi)
    mh = _log_int(rng, 1, 64)
    return _case(None, "paper", _log_int(rng, 1, min(64, max(1, 340000 // hi))), f"{lo}-{hi}", f"1-{mh}", shape=shape)


def _pair(text):
    lo, hi = text.split("-")
    return int(lo), int(hi)


def _shapes(case):
    """(history lengths, target counts) of the case's requests."""
    rng = np.random.default_rng([17, case["shape"]])
    R = case["requests"]
    lo, hi = _pair(case["L"])
    if case["sl"]:
        # L = L_min + s (L_max - L_min), s ~ Beta with mean l_avg, to a multiple of 8
        beta = SL_ALPHA * (hi - lo) / (lo - SL_MIN)
        L = SL_MIN + rng.beta(SL_ALPHA, beta, R) * (hi - SL_MIN)
        L = np.clip(np.round(L / 8) * 8, SL_MIN, hi).astype(np.int64)
        cap = hi  # the token budget: the longest are cut to one common length
        while np.minimum(L, cap).sum() > R * lo:
            cap -= 8
        L = np.minimum(L, cap)
    else:
        L = rng.integers(lo, hi, R, endpoint=True)
    mlo, mhi = _pair(case["m"])
    return L.astype(np.int64), rng.integers(mlo, mhi, R, endpoint=True).astype(np.int64)


def _offsets(counts):
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)


def _inputs(case, seed):
    """Rows, weights and upstream gradient on the GPU, in the storage type."""
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    L, m = _shapes(case)
    d, n, F = case["d"], case["layers"], FFN_MULT * case["d"]

    def normal(*shape, fan=1):
        return (torch.randn(*shape, generator=gen, device="cuda") / math.sqrt(fan)).to(dt)
    x = {"hist": normal(int(L.sum()), d), "tgt": normal(int(m.sum()), d)}
    for k in ("wq", "wk", "wv", "wo"):
        x[k] = normal(n, d, d, fan=d)
    if case["kind"] == "paper":
        x["ffn_u"], x["ffn_v"], x["ffn_o"] = normal(n, d, F, fan=d), normal(n, d, F, fan=d), normal(n, F, d, fan=F)
        x["wc"] = torch.cat([normal(k * d, d, fan=k * d) for k in range(2, n + 1)])
        x["wz"] = normal((n + 1) * d, d, fan=(n + 1) * d)
        x["z_u"], x["z_v"], x["z_o"] = normal(d, F, fan=d), normal(d, F, fan=d), normal(F, d, fan=F)
    else:
        x["w1"], x["w2"] = normal(n, d, F, fan=d), normal(n, F, d, fan=F)
    if case["kind"] == "train":
        x["dout"] = normal(int(m.sum()), d)
    return x, L, m


def prepare(case, seed):
    x, L, m = _inputs(case, seed)
    if case["kind"] == "paper":
        return _prepare_paper(case, x, L, m)
    wl = Workload("case", case["requests"], case["d"], case["heads"], case["layers"], case["dtype"], seed=0,
                  backward=case["kind"] == "train", ffn_mult=FFN_MULT)
    weights = {k: x[k] for k in ("wq", "wk", "wv", "wo", "w1", "w2")}
    b = Batch(wl, np.arange(len(L)), L, m, _offsets(L), _offsets(m), None, None, weights)
    db = DeviceBatch.from_tensors(b, x["hist"], x["tgt"], weights, backward=case["kind"] == "train")
    return {"kind": case["kind"], "db": db, "dout": x.get("dout")}


def _prepare_paper(case, x, L, m):
    hoff, toff = _offsets(L), _offsets(m)
    dev = {"hoff": torch.from_numpy(hoff).cuda(), "toff": torch.from_numpy(toff).cuda()}
    dims = stca.dims(case["d"], case["heads"], case["layers"], FFN_MULT * case["d"],
                     stca.STCA_BF16 if case["dtype"] == "bf16" else stca.STCA_F32)
    batch = stca.batch(len(L), int(hoff[-1]), int(toff[-1]), dev["hoff"], dev["toff"], hoff, toff)
    size = stca.stca_paper_workspace_size(dims, batch)
    return {"kind": "paper", "dims": dims, "batch": batch, "x": x, "keep": (hoff, toff, dev),
            "w": stca.paper_weights(**{k: x[k] for k in stca.PAPER_WEIGHT_FIELDS}),
            "z": torch.empty_like(x["tgt"]), "ws": torch.empty(size, dtype=torch.uint8, device="cuda"),
            "ws_bytes": size}


def run(state):
    if state["kind"] == "paper":
        stca.stca_forward_paper(state["dims"], state["batch"], state["x"]["hist"], state["x"]["tgt"], state["w"],
                                state["z"], None, state["ws"], state["ws_bytes"],
                                torch.cuda.current_stream().cuda_stream)
        return {"z": state["z"]}
    db = state["db"]
    if state["kind"] == "score":
        return {"out": db.forward()}
    # a training step: with the record where the batch has one, else the
    # forward and the backward that recomputes it
    record = db.record is not None
    out = db.forward_train() if record else db.forward()
    return {"out": out, **db.backward(state["dout"], use_record=record)}


def work(case):
    """The cheaper of the two evaluation orders for each request, the target
    side, and each input and output once; a training step's backward counts
    twice its forward."""
    L, m = _shapes(case)
    d, h, n, F = case["d"], case["heads"], case["layers"], FFN_MULT * case["d"]
    size = 2 if case["dtype"] == "bf16" else 4
    rows, tgts = int(L.sum()), int(m.sum())
    attn = float(np.minimum(4.0 * L * d * d + 4.0 * m * L * d, 4.0 * m * h * L * d).sum())
    flops = n * (attn + tgts * (4.0 * d * d + 4.0 * d * F))
    weights = n * (4 * d * d + 2 * d * F)
    nbytes = size * (rows * d + 2 * tgts * d + weights)
    if case["kind"] == "paper":
        extra = sum(k * d * d for k in range(2, n + 2)) + 3 * d * F
        weights = n * (4 * d * d + 3 * d * F) + extra
        flops = n * (attn + 6.0 * d * F * (rows + tgts)) + 2.0 * tgts * (n * 2 * d * d + extra)
        nbytes = size * (rows * d + 2 * tgts * d + weights)
    if case["kind"] == "train":
        flops *= 3
        nbytes += 4 * (rows * d + tgts * d + weights) + size * tgts * d
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # four times the largest error against exact() that was measured: 1.7e-3
    # on bf16 outputs (their own rounding, 2^-9), up to 6.4e-3 on gradients
    # formed from bf16 operands (stochastic lengths), 8e-7 in fp32, where a
    # ReLU gate within the rounding of zero may also fall the other way
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 2e-2 if case["kind"] == "train" else 7e-3}


def _attend(q, K, V, L, m, heads):
    """Every target's single query per head over its request's rows."""
    d = q.shape[1]
    dh = d // heads
    L, m = [int(v) for v in L], [int(v) for v in m]
    a = []
    for qr, kr, vr in zip(q.split(m), K.split(L), V.split(L)):
        qh = qr.view(-1, heads, dh).transpose(0, 1)
        kh = kr.view(-1, heads, dh).transpose(0, 1)
        vh = vr.view(-1, heads, dh).transpose(0, 1)
        p = torch.softmax(torch.matmul(qh, kh.transpose(1, 2)) / math.sqrt(dh), dim=-1)
        a.append(torch.matmul(p, vh).transpose(0, 1).reshape(-1, d))
    return torch.cat(a)


def _stack(x, L, m, heads):
    s = x["tgt"]
    for i in range(x["wq"].shape[0]):
        a = _attend(s @ x["wq"][i], x["hist"] @ x["wk"][i], x["hist"] @ x["wv"][i], L, m, heads)
        u = s + a @ x["wo"][i]
        s = u + torch.relu(u @ x["w1"][i]) @ x["w2"][i]
    return s


def _swiglu(x, wu, wv, wo):
    g = x @ wv
    return ((x @ wu) * (g * torch.sigmoid(g))) @ wo


def _paper_stack(x, L, m, heads):
    d, n = x["tgt"].shape[1], x["wq"].shape[0]

    def block(r, i):
        out = [_swiglu(c, x["ffn_u"][i], x["ffn_v"][i], x["ffn_o"][i]) for c in r.split(1 << 17)]
        return torch.nn.functional.layer_norm(torch.cat(out), (d,), eps=LN_EPS)
    outs, row, t = [], 0, x["tgt"]
    q = block(t, 0)
    for i in range(n):
        xt = block(x["hist"], i)
        outs.append(_attend(q @ x["wq"][i], xt @ x["wk"][i], xt @ x["wv"][i], L, m, heads) @ x["wo"][i])
        if i + 1 < n:
            k = (i + 2) * d
            q = block(torch.cat([*outs, t], dim=1) @ x["wc"][row:row + k], i + 1)
            row += k
    return _swiglu(torch.cat([*outs, t], dim=1) @ x["wz"], x["z_u"], x["z_v"], x["z_o"])


def exact(case, seed):
    x, L, m = _inputs(case, seed)
    x = {k: v.double() for k, v in x.items()}
    with torch.set_grad_enabled(case["kind"] == "train"):
        if case["kind"] == "paper":
            return {"z": _paper_stack(x, L, m, case["heads"])}
        if case["kind"] == "score":
            return {"out": _stack(x, L, m, case["heads"])}
        names = ("hist", "tgt", "wq", "wk", "wv", "wo", "w1", "w2")
        for k in names:
            x[k].requires_grad_()
        out = _stack(x, L, m, case["heads"])
        grads = torch.autograd.grad(out, [x[k] for k in names], x["dout"])
        return {"out": out.detach(), **{"d" + k: g for k, g in zip(names, grads)}}
