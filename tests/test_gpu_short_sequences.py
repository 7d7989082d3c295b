"""Short sequences that go through alone: every workgroup takes the state through the tiles before (backward: after) its own,
and the backward walk takes single tiles of a state cache that holds one state per pair. Lengths around the tiles and around
the longest that goes this way, odd and even tile counts, one more head than there are CUs for, against the brute-force
oracle at the tolerances of the other parity tests (1e-4 / 2e-2)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [("bf16", 128, 2, N) for N in (64, 65, 128, 129, 200, 256, 511, 512, 513)] + \
        [("bf16", 64, 3, N) for N in (127, 192, 320, 512)] + [("bf16", 128, 33, 512), ("bf16", 128, 86, 192)] + \
        [("f32", D, 2, N) for D in (64, 128) for N in (32, 33, 97, 128, 129)]


@pytest.mark.parametrize("token", [False, True])
@pytest.mark.parametrize("dtype,D,H,N", CASES)
def test_short_alone(oracle, dtype, D, H, N, token):
    from paper_2404_02882_amd import harness
    from paper_2404_02882_amd import synth_inputs as si
    print(f"case short dtype={dtype} D={D} H={H} N={N} token={token}", flush=True)
    inp = si.make_inputs(si.Config("short", B=1, H=H, N=N, D=D, chunk=64, dtype=dtype, seed=N + H, token_decay=token), with_states=True)
    rng = np.random.default_rng(N)
    if token:
        inp.log_g = np.log(rng.uniform(0.9, 1.0, (1, H, N))).astype(np.float32)
        o, kvo = oracle.gated_fwd_brute(inp.q, inp.k, inp.v, inp.log_g, inp.kv_in)
        dq, dk, dv, dlg, gin = oracle.gated_bwd_brute(inp.q, inp.k, inp.v, inp.dout, inp.log_g, inp.kv_in, inp.dkv_out)
        ref = dict(out=o, kv_out=kvo, dq=dq, dk=dk, dv=dv, dlog_g=dlg, dkv_in=gin)
    else:
        inp.decay = rng.uniform(0.95, 1.0, H).astype(np.float32)
        o, kvo = oracle.fwd_brute(inp.q, inp.k, inp.v, inp.decay, inp.kv_in)
        dq, dk, dv, gin = oracle.bwd_brute(inp.q, inp.k, inp.v, inp.dout, inp.decay, inp.kv_in, inp.dkv_out)
        ref = dict(out=o, kv_out=kvo, dq=dq, dk=dk, dv=dv, dkv_in=gin)
    tol = 1e-4 if dtype == "f32" else 2e-2
    for recompute in (False, True):
        got = harness.run_gpu(inp, recompute=recompute)
        for name, r in ref.items():
            emax, efro = harness.rel_errors(got[name], r)
            assert np.isfinite(emax) and emax <= tol and efro <= tol, (recompute, name, emax, efro)


@pytest.mark.parametrize("D,Dv", [(64, 64), (128, 128), (64, 128), (128, 64)])
@pytest.mark.parametrize("N", [64, 97, 100, 128])
def test_float_start_states_are_the_scanned_ones(N, D, Dv):
    """Float, one lambda per head: the states that workgroups compute themselves are to the last bit those of a local pass and
    a scan over as many segments (segments = tiles)."""
    from paper_2404_02882_amd import harness
    from paper_2404_02882_amd import synth_inputs as si
    print(f"case own start states N={N} {D}x{Dv}", flush=True)
    inp = si.make_inputs(si.Config("own", B=1, H=8, N=N, D=D, chunk=64, dtype="f32", seed=N + Dv, Dv=Dv), with_states=True)
    inp.decay = np.random.default_rng(N).uniform(0.95, 1.0, 8).astype(np.float32)
    got = [harness.run_gpu(inp, segments=s) for s in (0, -(-N // 32))]
    for name in ("out", "kv_out", "dq", "dv", "dkv_in"):
        assert np.array_equal(got[0][name], got[1][name]), name
    # (the waves that make dK keep the state the other way round and weigh q instead of dO: two roundings of 2^-24 a product apart)
    assert max(harness.rel_errors(got[0]["dk"], got[1]["dk"])) <= 1e-6


# Float forward calls without a cache, up to 256 tokens (k_short): edges of its 32-token tiles, the smallest and largest lengths that
# take it, one token more, with and without an entering state, grouped heads, one tile whose state wave is the last or the first.
@pytest.mark.parametrize("N", [13, 31, 32, 33, 64, 95, 223, 224, 255, 256, 257])
@pytest.mark.parametrize("D,kv_heads,states", [(64, 0, True), (64, 2, False), (128, 0, True), (128, 0, False)])
def test_short_float_forward(oracle, N, D, kv_heads, states):
    import torch
    from paper_2404_02882_amd import harness, lasp
    from paper_2404_02882_amd import synth_inputs as si
    cfg = si.Config("short", B=2, H=4, N=N, D=D, chunk=64, dtype="f32", seed=9700 + N + D)
    inp = si.make_inputs(cfg, with_states=True)
    G = 4 // kv_heads if kv_heads else 1
    k, v = inp.k[:, ::G].copy(), inp.v[:, ::G].copy()
    print(f"case N={N} D={D} kv_heads={kv_heads} states={states}", flush=True)
    shape = lasp.make_shape(2, 4, N, D, 64, "f32", kv_heads=kv_heads)
    dev = lambda x: torch.from_numpy(x).cuda()   # noqa: E731
    q, kd, vd = (harness.to_device(x, "f32") for x in (inp.q, k, v))
    out = torch.full_like(q, float("nan"))
    kv_out = torch.full((2, 4, D, D), float("nan"), device="cuda")
    scratch = torch.full((lasp.scratch_bytes(shape),), 0x7f, dtype=torch.uint8, device="cuda")
    lasp.lasp_fwd(shape, q, kd, vd, dev(inp.kv_in) if states else None, dev(inp.decay), out, kv_out, None, scratch)
    ref = oracle.dims_fwd_brute(inp.q, oracle.group_expand(k, G), oracle.group_expand(v, G), inp.decay, inp.kv_in if states else np.zeros_like(inp.kv_in))
    for name, x, r in zip(("out", "kv_out"), (out, kv_out), ref):
        emax, efro = harness.rel_errors(x.cpu().numpy(), r)
        print(f"  {name:7s} max-rel {emax:.3e} fro-rel {efro:.3e}", flush=True)
        assert np.isfinite(emax) and emax <= 1e-5 and efro <= 1e-6, name   # fp32 sums of at most 256 terms: 256^0.5 2^-24


@pytest.mark.parametrize("D,N", [(64, 100), (128, 256)])
def test_short_float_forward_keeps_the_entering_state(D, N):
    """A sequence object without a backward pass: the copy of the entering state comes with the launch."""
    import torch
    from paper_2404_02882_amd.sequence import LaspSequence
    g = torch.Generator(device="cuda").manual_seed(N)
    new = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    q, k, v, kv_in = new(1, 4, N, D), new(1, 4, N, D), new(1, 4, N, D), new(1, 4, D, D)
    seq = LaspSequence(1, 4, N, D, 64, torch.float32, need_backward=False)
    seq.kv[0].fill_(float("nan"))
    print(f"case kv copy D={D} N={N}", flush=True)
    seq.forward([q], [k], [v], torch.full((4,), 0.97, device="cuda"), [torch.empty_like(q)], kv_in)
    assert torch.equal(seq.kv[0], kv_in)
