"""Timing cases of the library: what its callers have it do, through the package's public entry points.

A case is a dict of plain values. `prepare` makes what a caller's program holds before the call (inputs, output
buffers, the sequence object with its workspace, a captured graph where the case uses one), `run` is one pass,
`work` the bytes and flops a pass cannot do without, `exact` the same results in 64 bits by plain torch.

Keys of a case (missing = 0 / False):
    kind        "train" forward + backward, "forward" forward only, "step" a few new tokens onto a carried state,
                "bidir" forward + backward without the causal mask
    dtype       "bf16" or "f32"
    B, H, N, D  batch, heads, tokens of the whole sequence, key dimension
    Dv          value dimension when it is not D
    T           sub-sequences the sequence is processed in
    kv_heads    key/value heads when fewer than H
    token       a decay per token (log g) instead of one lambda per head
    norm        outputs normalised row by row
    states      a state enters from the left (and, in a train case, a state gradient from the right)
    recompute   no state cache between the passes
    graph       the step is captured in a HIP graph once and replayed
    outliers    1 % of the key rows are eight times as large
"""
import math

import torch

from paper_2404_02882_amd import lasp
from paper_2404_02882_amd.sequence import BidirSequence, GraphedStep, LaspSequence

CHUNK = 128          # valid for every shape; the kernels' tile does not depend on it
NORM_EPS = 1e-5
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest call: a short float prompt, forward only; all launch and latency
        {"name": "short_f32_forward", "kind": "forward", "dtype": "f32", "B": 1, "H": 2, "N": 256, "D": 64},
        # generation: one new token for a batch of sequences, each continuing its own carried state
        {"name": "one_token", "kind": "step", "dtype": "bf16", "B": 8, "H": 16, "N": 1, "D": 128, "states": True},
        # many short sub-sequences with the state handed on, the loop captured in a graph as short shards ask for
        {"name": "short_shards_graph", "kind": "train", "dtype": "bf16", "B": 2, "H": 8, "N": 4096, "D": 64, "T": 4, "graph": True},
        # a training batch whose length is no multiple of anything, continuing a sequence
        {"name": "ragged_train", "kind": "train", "dtype": "bf16", "B": 2, "H": 16, "N": 5000, "D": 128, "states": True},
        # the headline: one long sequence, 16 heads
        {"name": "long_train", "kind": "train", "dtype": "bf16", "B": 1, "H": 16, "N": 32768, "D": 128},
        # the largest: a batch of long sequences, 128 head chains, heavy-tailed keys
        {"name": "many_heads_train", "kind": "train", "dtype": "bf16", "B": 4, "H": 32, "N": 16384, "D": 128, "outliers": True},
        # the same long sequence with data-dependent decay (and its gradient)
        {"name": "token_decay_train", "kind": "train", "dtype": "bf16", "B": 1, "H": 16, "N": 32768, "D": 128, "token": True},
        # with the output normalisation fused
        {"name": "norm_train", "kind": "train", "dtype": "bf16", "B": 1, "H": 16, "N": 32768, "D": 128, "norm": True},
        # with keys narrower than values
        {"name": "narrow_keys_train", "kind": "train", "dtype": "bf16", "B": 1, "H": 16, "N": 32768, "D": 64, "Dv": 128},
        # without mask and decay: an encoder
        {"name": "bidirectional_train", "kind": "bidir", "dtype": "bf16", "B": 1, "H": 16, "N": 32768, "D": 128},
        # full precision training, for reference runs and debugging
        {"name": "f32_train", "kind": "train", "dtype": "f32", "B": 1, "H": 16, "N": 8192, "D": 128},
        # grouped key/value heads, two sub-sequences
        {"name": "grouped_heads_train", "kind": "train", "dtype": "bf16", "B": 1, "H": 32, "N": 8192, "D": 128, "T": 2, "kv_heads": 4},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["train", "forward", "step", "bidir"], [60, 15, 10, 15])[0]
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    c = {"kind": kind, "dtype": dtype, "D": rng.choice([128, 128, 64])}
    c["B"], c["H"] = rng.choice([(1, 2), (1, 8), (2, 8), (1, 16), (2, 16), (1, 32), (8, 16), (4, 32)])
    if kind == "step":
        c["N"] = _log_uniform(rng, 1, 64)
        c["states"] = True
        c["token"] = rng.random() < 0.3
        return c
    # tokens of one sub-sequence: over the whole range, no multiple of any tile in two draws of five
    most = (131072 if dtype == "f32" else 1048576) // (c["B"] * c["H"])
    n = _log_uniform(rng, 64, min(32768, most))
    if rng.random() < 0.6:
        n = max(64, n // 128 * 128)
    c["T"] = rng.choice([t for t in (1, 1, 1, 2, 4) if n * t <= most] or [1])
    c["N"] = n * c["T"]
    if kind == "bidir":
        return c
    c["token"] = rng.random() < 0.25
    c["norm"] = rng.random() < 0.2
    c["states"] = rng.random() < 0.4
    if rng.random() < 0.15:
        c["D"], c["Dv"] = rng.choice([(64, 128), (128, 64)])
    if rng.random() < 0.2 and c["H"] >= 8:
        c["kv_heads"] = c["H"] // rng.choice([2, 4, 8])
    if kind == "train":
        c["recompute"] = rng.random() < 0.15
        c["graph"] = rng.random() < 0.2
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _sizes(case):
    B, H, N, D = (case[x] for x in ("B", "H", "N", "D"))
    return B, H, N, D, case.get("Dv") or D, case.get("T") or 1, case.get("kv_heads") or H


def _decay_schedule(H, device):
    """lambda_h = 1 - 2^-(5 + 8 h / H), as float32."""
    h = torch.arange(H, dtype=torch.float64, device=device)
    return (1.0 - torch.exp2(-(5.0 + 8.0 * h / H))).float()


def _inputs(case, seed, device="cuda"):
    """The whole sequence's tensors, made from the seed alone: q, k, v as a layer's projections give them (N(0,1)
    over the root of the dimension), dO ~ N(0,1), states ~ N(0,1), log g around the heads' fixed rates with one
    token in a thousand almost closing the gate."""
    B, H, N, D, Dv, T, KH = _sizes(case)
    dt = DTYPES[case["dtype"]]
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))

    def normal(*shape, scale=1.0):
        return torch.randn(*shape, generator=g, device=device, dtype=torch.float32) * scale

    x = {}
    x["q"] = normal(B, H, N, D, scale=D ** -0.5).to(dt)
    k = normal(B, KH, N, D, scale=D ** -0.5)
    if case.get("outliers"):
        k = torch.where(torch.rand(B, KH, N, 1, generator=g, device=device) < 0.01, k * 8.0, k)
    x["k"] = k.to(dt)
    x["v"] = normal(B, KH, N, Dv, scale=Dv ** -0.5).to(dt)
    if case["kind"] in ("train", "bidir"):
        x["dout"] = normal(B, H, N, Dv).to(dt)
    lam = _decay_schedule(H, device)
    if case.get("token"):
        lg = lam.double().log()[None, :, None] * 2.0 * torch.rand(B, H, N, generator=g, device=device, dtype=torch.float64)
        closed = torch.rand(B, H, N, generator=g, device=device) < 0.001
        x["log_g"] = torch.where(closed, torch.full_like(lg, -8.0), lg).float()
    else:
        x["decay"] = lam
    if case.get("states"):
        x["kv_in"] = normal(B, H, D, Dv)
        if case["kind"] == "train":
            x["dkv_out"] = normal(B, H, D, Dv)
    return x


def _shards(x, T):
    return [s.contiguous() for s in x.chunk(T, dim=2)]


def prepare(case, seed):
    B, H, N, D, Dv, T, KH = _sizes(case)
    dt, kind = DTYPES[case["dtype"]], case["kind"]
    x = _inputs(case, seed)
    s = {"case": case}
    if kind == "step":
        token = bool(case.get("token"))
        shape = lasp.make_shape(B, H, N, D, CHUNK, dt)
        size = lasp.gated_scratch_bytes(shape) if token else lasp.scratch_bytes(shape)
        s.update(shape=shape, scratch=torch.empty(size, dtype=torch.uint8, device="cuda"), out=torch.empty_like(x["v"]),
                 kv_out=torch.empty_like(x["kv_in"]), decay=x["log_g"] if token else x["decay"], q=x["q"], k=x["k"], v=x["v"],
                 kv_in=x["kv_in"])
        return s
    q, k, v = (_shards(x[name], T) for name in ("q", "k", "v"))
    out = [torch.empty(B, H, N // T, Dv, dtype=dt, device="cuda") for _ in range(T)]
    if kind == "bidir":
        seq = BidirSequence(B, H, [N // T] * T, D, CHUNK, dt)
    else:
        seq = LaspSequence(B, H, N, D, CHUNK, dt, T=T, need_backward=kind == "train", token_decay=bool(case.get("token")),
                           norm_eps=NORM_EPS if case.get("norm") else None, kv_heads=case.get("kv_heads") or 0,
                           Dv=case.get("Dv") or 0, recompute=bool(case.get("recompute")))
    fwd = {"q": q, "k": k, "v": v, "out": out}
    rstd = dlog_g = None
    if kind != "bidir":
        fwd["decay"] = _shards(x["log_g"], T) if case.get("token") else x["decay"]
        fwd["kv_in"] = x.get("kv_in")
        if case.get("norm"):
            rstd = [torch.empty(B, H, N // T, device="cuda") for _ in range(T)]
        fwd["rstd"] = rstd
    s.update(seq=seq, fwd=fwd, out=out, rstd=rstd)
    if kind != "forward":
        dq = [torch.empty_like(t) for t in q]
        dk, dv = [torch.empty_like(t) for t in k], [torch.empty_like(t) for t in v]
        bwd = {"q": q, "k": k, "v": v, "dout": _shards(x["dout"], T), "dq": dq, "dk": dk, "dv": dv}
        if kind == "train":
            if case.get("token"):
                dlog_g = [torch.empty_like(t) for t in fwd["decay"]]
            bwd.update(decay=fwd["decay"], dkv_out=x.get("dkv_out"), dlog_g=dlog_g, out=out if case.get("norm") else None, rstd=rstd)
        s.update(bwd=bwd, dq=dq, dk=dk, dv=dv, dlog_g=dlog_g)
    if case.get("graph"):
        s["graph"] = GraphedStep(seq, fwd, s.get("bwd"))
    return s


def run(state):
    kind = state["case"]["kind"]
    if kind == "step":
        step = lasp.lasp_gated_fwd if state["case"].get("token") else lasp.lasp_fwd
        if state["case"].get("token"):
            step(state["shape"], state["q"], state["k"], state["v"], state["decay"], state["kv_in"], state["out"],
                 state["kv_out"], None, state["scratch"])
        else:
            step(state["shape"], state["q"], state["k"], state["v"], state["kv_in"], state["decay"], state["out"],
                 state["kv_out"], None, state["scratch"])
        return {"out": [state["out"]], "kv_out": state["kv_out"]}
    seq, got = state["seq"], {"out": state["out"]}
    if "graph" in state:
        state["graph"].replay()
        kv, dkv = seq.kv[seq.T], seq.dkv[0]
    else:
        kv = seq.forward(**state["fwd"])
        dkv = seq.backward(**state["bwd"]) if kind != "forward" else None
    got["kv_out"] = kv
    if state["rstd"] is not None:
        got["rstd"] = state["rstd"]
    if kind != "forward":
        got.update(dq=state["dq"], dk=state["dk"], dv=state["dv"], dkv_in=dkv)
        if state["dlog_g"] is not None:
            got["dlog_g"] = state["dlog_g"]
    return got


def work(case):
    """Every input read once and every output written once; the products of the recurrent form (state update and
    read-out forward; both state recurrences' read-outs and the gradient state's update backward)."""
    B, H, N, D, Dv, T, KH = _sizes(case)
    e = 2 if case["dtype"] == "bf16" else 4
    q, v, k_, v_ = B * H * N * D * e, B * H * N * Dv * e, B * KH * N * D * e, B * KH * N * Dv * e
    row, state = B * H * N * 4, B * H * D * Dv * 4
    nbytes = q + k_ + v_ + v + state            # forward: q, k, v, out, kv_out
    flops = 4 * B * H * N * D * Dv
    if case.get("states"):
        nbytes += state
    if case.get("token"):
        nbytes += row
    if case.get("norm"):
        nbytes += row
    if case["kind"] in ("train", "bidir"):      # q, k, v, dout, dq, dk, dv, dkv_in
        nbytes += 2 * q + 2 * k_ + 2 * v_ + v + state
        flops += 8 * B * H * N * D * Dv
        if case.get("states"):
            nbytes += state
        if case.get("token"):                   # log g, dlog g
            nbytes += 2 * row
        if case.get("norm"):                    # y, rstd
            nbytes += v + row
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the distance to `exact` measured over the listed cases and 340 drawn ones. bf16 (operands and
    outputs rounded to 8 bits): at most 3.3e-3, single values 0.039 of the root mean square. f32: at most 7.1e-7 and
    6.4e-6. The gradient of a per-token decay is a sum over the whole tail in which most of q.dq - k.dk cancels:
    0.026 and 0.10 in bf16, 1.4e-6 in f32."""
    if case["dtype"] == "f32":
        return {"rel": 6e-6 if case.get("token") else 3e-6, "max": 3e-5}
    if case.get("token") and case["kind"] == "train":
        return {"rel": 3e-2, "max": 0.4}
    return {"rel": 1.3e-2, "max": 0.15}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
def _chunks(N, C=128):
    return [(a, min(a + C, N)) for a in range(0, N, C)]


def _weights(lg):
    """Of a chunk with log decays lg [.., n]: weight of key j at query i, of the entering state at query i, of key j
    at the chunk's end, and of the entering state at the chunk's end."""
    cum = lg.cumsum(-1)
    n = lg.shape[-1]
    diff = cum[..., :, None] - cum[..., None, :]
    mask = torch.ones(n, n, dtype=torch.bool, device=lg.device).tril()
    M = torch.where(mask, diff, torch.full_like(diff, -math.inf)).exp()
    return M, cum.exp()[..., :, None], (cum[..., -1:] - cum).exp()[..., :, None], cum[..., -1:].exp()[..., None]


def exact(case, seed):
    B, H, N, D, Dv, T, KH = _sizes(case)
    x = _inputs(case, seed)
    d = lambda t: t.double()   # noqa: E731
    rep = H // KH
    q = d(x["q"])
    k, v = (d(x[n]).repeat_interleave(rep, dim=1) if rep > 1 else d(x[n]) for n in ("k", "v"))
    if case["kind"] == "bidir":
        do = d(x["dout"])
        kv, dkv = k.transpose(-1, -2) @ v, q.transpose(-1, -2) @ do
        return {"out": _shards(q @ kv, T), "kv_out": kv, "dq": _shards(do @ kv.transpose(-1, -2), T),
                "dk": _shards(v @ dkv.transpose(-1, -2), T), "dv": _shards(k @ dkv, T), "dkv_in": dkv}
    lg = d(x["log_g"]) if case.get("token") else d(x["decay"]).log()[None, :, None].expand(B, H, N)
    zero = torch.zeros(B, H, D, Dv, dtype=torch.float64, device=q.device)
    kv = d(x["kv_in"]) if "kv_in" in x else zero
    out, entering = torch.empty_like(v), []
    for a, b in _chunks(N):
        M, up, after, whole = _weights(lg[:, :, a:b])
        Q, K, V = q[:, :, a:b], k[:, :, a:b], v[:, :, a:b]
        entering.append(kv)
        out[:, :, a:b] = ((Q @ K.transpose(-1, -2)) * M) @ V + up * (Q @ kv)
        kv = whole * kv + (after * K).transpose(-1, -2) @ V
    kv_out = kv
    got = {"kv_out": kv_out}
    if case.get("norm"):
        rstd = (out.square().mean(-1) + NORM_EPS).rsqrt()
        y = out * rstd[..., None]
        got.update(out=_shards(y, T), rstd=_shards(rstd, T))
    else:
        got["out"] = _shards(out, T)
    if case["kind"] != "train":
        return got
    do = d(x["dout"])
    if case.get("norm"):
        do = rstd[..., None] * (do - y * (do * y).mean(-1, keepdim=True))
    dkv = d(x["dkv_out"]) if "dkv_out" in x else zero
    edge = (dkv * kv_out).sum((-1, -2))
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    for (a, b), kv in zip(reversed(_chunks(N)), reversed(entering)):
        M, up, after, whole = _weights(lg[:, :, a:b])
        Q, K, V, G = q[:, :, a:b], k[:, :, a:b], v[:, :, a:b], do[:, :, a:b]
        S, dS = (Q @ K.transpose(-1, -2)) * M, (G @ V.transpose(-1, -2)) * M
        dq[:, :, a:b] = dS @ K + up * (G @ kv.transpose(-1, -2))
        dk[:, :, a:b] = dS.transpose(-1, -2) @ Q + after * (V @ dkv.transpose(-1, -2))
        dv[:, :, a:b] = S.transpose(-1, -2) @ G + after * (K @ dkv)
        dkv = whole * dkv + (up * Q).transpose(-1, -2) @ G
    if case.get("token"):   # d log g_s = <dkv_out, kv_out> + sum over t >= s of (q_t . dq_t - k_t . dk_t)
        r = (q * dq - k * dk).sum(-1)
        got["dlog_g"] = _shards(edge[..., None] + r.flip(-1).cumsum(-1).flip(-1), T)
    if rep > 1:
        dk, dv = (t.unflatten(1, (KH, rep)).sum(2) for t in (dk, dv))
    got.update(dq=_shards(dq, T), dk=_shards(dk, T), dv=_shards(dv, T), dkv_in=dkv)
    return got
