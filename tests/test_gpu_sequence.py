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
def test_together(gpu, oracle, dtype, D, Dv, n, T, kv_heads, token, norm, recompute, H=4):
    harness, lasp, sequence, si = gpu
    N, G = n * T, H // kv_heads if kv_heads else 1
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


# (H, data type, D, Dv, tokens, T): sub-sequences whose last segment is short and has several tiles of the local pass (which cuts
# it from its end: three of 128 tokens, three of 64 where d_k is not d_v, two of 32), and sequences whose last group is one
# sub-sequence with a plan of its own (4, 4, 4, 1 and 2, 1)
LONGER = [(32, "bf16", 128, 0, 1050, 2), (32, "bf16", 128, 64, 1180, 2), (32, "f32", 128, 0, 1000, 2),
          (4, "bf16", 128, 0, 130, 13), (4, "f32", 64, 0, 40, 13), (100, "bf16", 64, 0, 130, 3)]


@pytest.mark.parametrize("H,dtype,D,Dv,n,T", LONGER)
@pytest.mark.parametrize("recompute", [False, True])
def test_together_longer_segments_and_one_left_over(gpu, oracle, H, dtype, D, Dv, n, T, recompute):
    test_together(gpu, oracle, dtype, D, Dv, n, T, 0, False, False, recompute, H)


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


@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("D,n", [(64, 24576), (128, 1000)])
def test_decay_per_token_is_call_after_call(gpu, D, n, norm):
    """With a decay per token a sequence is what one call after the other computes, to the last bit: the gradient of log g is a
    sum over each sub-sequence's tail in which most cancels, and holds only for the states the walks themselves start from."""
    import torch
    harness, lasp, sequence, si = gpu
    B, H, T, eps, bf = 1, 2, 4, 1e-5, torch.bfloat16
    print(f"case call after call D={D} n={n} norm={norm}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    q, k, v, do = ([(rnd(B, H, n, D) * D ** -0.5).to(bf) for _ in range(T)] for _ in range(4))
    lg = [torch.rand(B, H, n, generator=g, device="cuda") * -1e-3 for _ in range(T)]
    kv_in, dkv_out = rnd(B, H, D, D), rnd(B, H, D, D)
    seq = sequence.LaspSequence(B, H, n * T, D, 64, bf, T=T, token_decay=True, norm_eps=eps if norm else None)
    fresh = lambda like: [torch.empty_like(x) for x in like]   # noqa: E731

    def by_sequence():
        out, dq, dk, dv, dlg = (fresh(x) for x in (v, q, k, v, lg))
        rstd = fresh(lg) if norm else None
        seq.forward(q, k, v, lg, out, kv_in, rstd)
        seq.backward(q, k, v, do, lg, dq, dk, dv, dkv_out, dlg, out if norm else None, rstd)
        return out + dq + dk + dv + dlg + seq.kv[1:] + seq.dkv[:T]

    def by_calls():
        out, rstd, dq, dk, dv, dlg = (fresh(x) for x in (v, lg, q, k, v, lg))
        kv, dkv = [kv_in] + fresh(seq.kv[1:]), fresh(seq.dkv[:T]) + [dkv_out]
        one = lasp.make_shape(B, H, n, D, 64, bf)
        scratch = torch.empty(lasp.gated_scratch_bytes(one), dtype=torch.uint8, device="cuda")
        caches = fresh(seq.caches)
        for t in range(T):
            if norm:
                lasp.lasp_gated_fwd_norm(one, q[t], k[t], v[t], lg[t], kv[t], eps, out[t], rstd[t], kv[t + 1], caches[t], scratch)
            else:
                lasp.lasp_gated_fwd(one, q[t], k[t], v[t], lg[t], kv[t], out[t], kv[t + 1], caches[t], scratch)
        for t in reversed(range(T)):
            if norm:
                lasp.lasp_gated_bwd_norm(one, q[t], k[t], v[t], out[t], rstd[t], do[t], lg[t], kv[t], kv[t + 1], dkv[t + 1], caches[t],
                                         dq[t], dk[t], dv[t], dlg[t], dkv[t], scratch)
            else:
                lasp.lasp_gated_bwd(one, q[t], k[t], v[t], do[t], lg[t], kv[t], kv[t + 1], dkv[t + 1], caches[t], dq[t], dk[t], dv[t], dlg[t],
                                    dkv[t], scratch)
        return out + dq + dk + dv + dlg + kv[1:] + dkv[:T]

    a, b = by_sequence(), by_calls()
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(a, b)) and all(torch.isfinite(x).all() for x in a)


@pytest.mark.parametrize("dtype,n", [("bf16", 256), ("f32", 100)])
def test_states_in_turn(gpu, dtype, n):
    """Two states written in turn (kv[0] = kv[2], kv[1] = kv[3]): the copy of the entering state goes to memory that the second
    sub-sequence writes, so the sequence goes one by one, to the last bit like sub-sequences with states of their own."""
    import torch
    harness, lasp, sequence, si = gpu
    B, H, D, T = 1, 3, 64, 3
    inp = si.make_inputs(si.Config("turn", B=B, H=H, N=n * T, D=D, chunk=64, dtype=dtype, seed=78), with_states=True)
    q, k, v, do = (harness.shards(x, T, dtype) for x in (inp.q, inp.k, inp.v, inp.dout))
    decay, kv_in, dkv_out = (torch.from_numpy(x).cuda() for x in (inp.decay, inp.kv_in, inp.dkv_out))
    fresh = lambda like: [torch.empty_like(x) for x in like]   # noqa: E731

    def run(in_turn):
        seq = sequence.LaspSequence(B, H, n * T, D, 64, harness.TORCH_DTYPE[dtype], T=T)
        out, dq, dk, dv = (fresh(x) for x in (v, q, k, v))
        if in_turn:
            for states in (seq.kv, seq.dkv):
                states[2:] = states[:2]
            seq.forward(q, k, v, decay, out, kv_in)
            seq.backward(q, k, v, do, decay, dq, dk, dv, dkv_out)
        else:
            one, entering, leaving = lasp.make_shape(B, H, n, D, 64, harness.TORCH_DTYPE[dtype]), [kv_in] + seq.kv[1:], seq.dkv[:T] + [dkv_out]
            for t in range(T):
                lasp.lasp_fwd(one, q[t], k[t], v[t], entering[t], decay, out[t], seq.kv[t + 1], seq.caches[t], seq.scratch)
            for t in reversed(range(T)):
                lasp.lasp_bwd(one, q[t], k[t], v[t], do[t], None, leaving[t + 1], decay, seq.caches[t], dq[t], dk[t], dv[t], seq.dkv[t], seq.scratch)
        torch.cuda.synchronize()
        return out + dq + dk + dv + [seq.kv[T], seq.dkv[0]]

    assert all(torch.equal(a, b) for a, b in zip(run(True), run(False)))
