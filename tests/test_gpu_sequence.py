"""Sub-sequences that go through a launch together (lasp_seq_fwd / lasp_seq_bwd), against the fp64 oracle and against one
call after the other. Tolerances 1e-4 float, 2e-2 bfloat16 as everywhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "needs a GPU"
    from paper_2404_02882_amd import harness, lasp, sequence, synth_inputs
    return harness, lasp, sequence, synth_inputs


# (data type, D, Dv, tokens of a sub-sequence, T, K/V heads, decay per token, Norm): whole tiles, short last tiles whose
# segments other sub-sequences start behind (the forward local pass cuts them from the end), odd numbers of 64-token tiles
# under its 128-token tiles, sub-sequences of less than a tile, more of them than a launch takes
CASES = [
    ("bf16", 64, 0, 256, 4, 0, False, False), ("bf16", 128, 0, 320, 3, 0, False, True), ("bf16", 128, 0, 333, 4, 2, False, False),
    ("bf16", 128, 0, 65, 2, 0, True, False), ("bf16", 64, 0, 5, 3, 0, False, False), ("bf16", 128, 64, 129, 2, 0, False, False),
    ("bf16", 64, 128, 192, 2, 2, True, True), ("bf16", 128, 0, 130, 9, 0, False, False), ("bf16", 64, 0, 447, 10, 0, True, False),
    ("f32", 64, 0, 70, 4, 0, False, False), ("f32", 128, 0, 33, 3, 2, False, True), ("f32", 128, 64, 95, 2, 0, True, False),
    ("f32", 64, 0, 31, 9, 0, True, True),
]


@pytest.mark.parametrize("dtype,D,Dv,n,T,kv_heads,token,norm", CASES)
@pytest.mark.parametrize("recompute", [False, True])
def test_together(gpu, oracle, dtype, D, Dv, n, T, kv_heads, token, norm, recompute):
    harness, lasp, sequence, si = gpu
    H, N, G = 4, n * T, 4 // kv_heads if kv_heads else 1
    cfg = si.Config("seq", B=1, H=H, N=N, D=D, chunk=64, dtype=dtype, seed=9100 + n + T, token_decay=token, Dv=Dv)
    inp = si.make_inputs(cfg, with_states=True)
    print(f"case {dtype} {D}x{Dv or D} {T} x {n} kv_heads={kv_heads} token={token} norm={norm} recompute={recompute}", flush=True)
    inp.k, inp.v = inp.k[:, ::G].copy(), inp.v[:, ::G].copy()
    k, v = oracle.group_expand(inp.k, G), oracle.group_expand(inp.v, G)
    decay = None if token else inp.decay
    eps = 1e-5 if norm else None
    got = harness.run_gpu(inp, T=T, norm_eps=eps, recompute=recompute)
    o, kvo = oracle.dims_fwd_brute(inp.q, k, v, decay, inp.kv_in, log_g=inp.log_g)
    dout = inp.dout
    if norm:
        o, rstd = oracle.norm_fwd(o, eps)
        dout = oracle.norm_bwd(inp.dout, o, rstd)
    g = oracle.dims_bwd_brute(inp.q, k, v, dout, decay, inp.kv_in, inp.dkv_out, log_g=inp.log_g)
    names = ("dq", "dk", "dv", "dkv_in") if len(g) == 4 else ("dq", "dk", "dv", "dlog_g", "dkv_in")
    ref = dict(zip(names, g), out=o, kv_out=kvo)
    ref["dk"], ref["dv"] = (oracle.group_reduce(ref[x], G) for x in ("dk", "dv"))
    for name, r in ref.items():
        emax, efro = harness.rel_errors(got[name], r)
        print(f"  {name:7s} max-rel {emax:.3e} fro-rel {efro:.3e}", flush=True)
        assert np.isfinite(emax) and emax <= TOL[dtype] and efro <= TOL[dtype], name


@pytest.mark.parametrize("dtype,n", [("bf16", 200), ("f32", 100)])
def test_states_between_and_buffers_that_overlap(gpu, oracle, dtype, n):
    """Every state between the sub-sequences is that of call after call; a sequence whose sub-sequences write to one output
    buffer, or whose entering state is one it writes, is taken one by one, or from a copy."""
    import torch
    harness, lasp, sequence, si = gpu
    B, H, D, T = 1, 3, 64, 3
    cfg = si.Config("seq2", B=B, H=H, N=n * T, D=D, chunk=64, dtype=dtype, seed=77)
    inp = si.make_inputs(cfg, with_states=True)
    dt = harness.TORCH_DTYPE[dtype]
    q, k, v, do = (harness.shards(x, T, dtype) for x in (inp.q, inp.k, inp.v, inp.dout))
    decay, kv_in, dkv_out = (torch.from_numpy(x).cuda() for x in (inp.decay, inp.kv_in, inp.dkv_out))

    def run(segments, out, entering=lambda s: (kv_in, dkv_out)):
        seq = sequence.LaspSequence(B, H, n * T, D, 64, dt, T=T, segments=segments)
        a, b = entering(seq)
        seq.forward(q, k, v, decay, out, a)
        dq, dk, dv = ([torch.empty_like(x) for x in y] for y in (q, k, v))
        seq.backward(q, k, v, do, decay, dq, dk, dv, b)
        torch.cuda.synchronize()
        host = lambda ts: [t.float().cpu().numpy() for t in ts]   # noqa: E731
        return host(seq.kv), host(seq.dkv), host(out), host(dq), host(dk), host(dv)

    fresh = lambda: [torch.empty_like(x) for x in v]   # noqa: E731
    single = run(1, fresh())   # (a number of segments of the caller's own: one call after the other)
    together = run(0, fresh())
    shared = fresh()[0]
    one_buffer = run(0, [shared] * T)

    def from_own(seq):   # states that the call itself writes
        seq.kv[T].copy_(kv_in)
        seq.dkv[0].copy_(dkv_out)
        return seq.kv[T], seq.dkv[0]
    own = run(0, fresh(), from_own)

    def strided(seq):    # not in one piece
        pair = torch.stack([kv_in, dkv_out], dim=-1)
        return pair[..., 0], pair[..., 1]
    pieces = run(0, fresh(), strided)
    for got, skip in ((together, None), (one_buffer, 2), (own, None), (pieces, None)):
        for i, (x, y) in enumerate(zip(got, single)):
            for a, b in zip(x, y):
                if i == skip:
                    a, b = x[-1], y[-1]   # the last sub-sequence's output is what stays in the buffer
                emax, efro = harness.rel_errors(a, b)
                assert emax <= TOL[dtype] and efro <= TOL[dtype], (i, emax, efro)
    assert all(np.array_equal(a, b) for x, y in zip(own, together) for a, b in zip(x, y))
