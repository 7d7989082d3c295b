"""The state cache serves a backward call with another `segments` than the forward call's (the cut into segments is
each call's own affair), against the fp64 oracle. Tolerances 1e-4 float, 2e-2 bfloat16 as everywhere."""
from dataclasses import replace

import numpy as np
import pytest

from test_sequence_launches import PIECES_OF_A_SHARD

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "needs a GPU"
    from paper_2404_02882_amd import harness, lasp, synth_inputs
    return harness, lasp, synth_inputs


@pytest.mark.parametrize("dtype,tile", [("f32", 32), ("bf16", 64)])
@pytest.mark.parametrize("D,Dv", [(64, 64), (128, 64)])
@pytest.mark.parametrize("token", [False, True])
@pytest.mark.parametrize("fwd_segments,bwd_segments", [(0, 2), (3, 0), (2, 5), (9, 1)])
def test_forward_and_backward_cut_differently(gpu, oracle, dtype, tile, D, Dv, token, fwd_segments, bwd_segments):
    import torch
    harness, lasp, si = gpu
    N = 9 * tile + 5
    cfg = si.Config("segments", B=1, H=3, N=N, D=D, chunk=64, dtype=dtype, seed=8300 + N + D, token_decay=token, Dv=Dv)
    inp = si.make_inputs(cfg, with_states=True)
    print(f"case {dtype} {D}x{Dv} token={token} segments {fwd_segments} -> {bwd_segments}", flush=True)
    q, k, v, do = (harness.to_device(x, dtype) for x in (inp.q, inp.k, inp.v, inp.dout))
    dev = lambda x: torch.from_numpy(x).cuda()   # noqa: E731
    decay, kv_in, dkv_out = dev(inp.log_g if token else inp.decay), dev(inp.kv_in), dev(inp.dkv_out)
    shape = {s: lasp.make_shape(1, 3, N, D, 64, dtype, segments=s, Dv=Dv) for s in (fwd_segments, bwd_segments)}
    cache_bytes, scratch_bytes = ((lasp.gated_state_cache_bytes, lasp.gated_scratch_bytes) if token else
                                  (lasp.state_cache_bytes, lasp.scratch_bytes))
    f, b = shape[fwd_segments], shape[bwd_segments]
    assert cache_bytes(f) == cache_bytes(b)   # the size does not depend on the segments
    cache = torch.full((cache_bytes(f),), 0x7f, dtype=torch.uint8, device="cuda")   # (a slot that is never written would show)
    scratch = torch.full((max(scratch_bytes(f), scratch_bytes(b)),), 0x7f, dtype=torch.uint8, device="cuda")
    out, kv_out, dkv_in = torch.empty_like(v), torch.empty_like(kv_in), torch.empty_like(kv_in)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    if token:
        dlg = torch.empty_like(decay)
        lasp.lasp_gated_fwd(f, q, k, v, decay, kv_in, out, kv_out, cache, scratch)
        lasp.lasp_gated_bwd(b, q, k, v, do, decay, kv_in, kv_out, dkv_out, cache, dq, dk, dv, dlg, dkv_in, scratch)
        ref = oracle.dims_bwd_brute(inp.q, inp.k, inp.v, inp.dout, None, inp.kv_in, inp.dkv_out, log_g=inp.log_g)
    else:
        lasp.lasp_fwd(f, q, k, v, kv_in, decay, out, kv_out, cache, scratch)
        lasp.lasp_bwd(b, q, k, v, do, kv_in, dkv_out, decay, cache, dq, dk, dv, dkv_in, scratch)
        ref = oracle.dims_bwd_brute(inp.q, inp.k, inp.v, inp.dout, inp.decay, inp.kv_in, inp.dkv_out)
    got = dict(dq=dq, dk=dk, dv=dv, dkv_in=dkv_in)
    ref = dict(zip(("dq", "dk", "dv", "dkv_in") if len(ref) == 4 else ("dq", "dk", "dv", "dlog_g", "dkv_in"), ref))
    if token:
        got["dlog_g"] = dlg
    for name, r in ref.items():
        emax, efro = harness.rel_errors(got[name].float().cpu().numpy(), r)
        print(f"  {name:7s} max-rel {emax:.3e} fro-rel {efro:.3e}", flush=True)
        assert np.isfinite(emax) and emax <= TOL[dtype] and efro <= TOL[dtype], name


# (tokens, segments): the backward walk's segments of an odd number of 64-token tiles begin and end inside a pair
@pytest.mark.parametrize("N,segments", [(64 * 7, 7), (64 * 7, 3), (64 * 3, 0), (64 * 5 + 1, 6), (64 * 6 - 1, 2), (64 * 9, 2), (64, 1), (65, 2)])
@pytest.mark.parametrize("D,Dv,kv_heads", [(64, 64, 0), (128, 128, 0), (128, 128, 2), (64, 128, 0), (128, 64, 0)])
@pytest.mark.parametrize("token,norm", [(False, False), (True, False), (False, True), (True, True)])
def test_odd_segments(gpu, oracle, N, segments, D, Dv, kv_heads, token, norm):
    harness, lasp, si = gpu
    cfg = si.Config("odd", B=1, H=4, N=N, D=D, chunk=64, dtype="bf16", seed=8500 + N + D, token_decay=token, Dv=Dv)
    inp = si.make_inputs(cfg, with_states=True)
    print(f"case N={N} segments={segments} {D}x{Dv} kv_heads={kv_heads} token={token} norm={norm}", flush=True)
    G = 4 // kv_heads if kv_heads else 1
    inp.k, inp.v = inp.k[:, ::G].copy(), inp.v[:, ::G].copy()
    k, v = oracle.group_expand(inp.k, G), oracle.group_expand(inp.v, G)
    decay = None if token else inp.decay
    eps = 1e-5 if norm else None
    got = harness.run_gpu(inp, segments=segments, norm_eps=eps)
    o, kvo = oracle.dims_fwd_brute(inp.q, k, v, decay, inp.kv_in, log_g=inp.log_g)
    dout = inp.dout
    if norm:
        o, rstd = oracle.norm_fwd(o, eps)
        dout = oracle.norm_bwd(inp.dout, o, rstd)
    g = oracle.dims_bwd_brute(inp.q, k, v, dout, decay, inp.kv_in, inp.dkv_out, log_g=inp.log_g)
    ref = dict(out=o, kv_out=kvo, dq=g[0], dk=oracle.group_reduce(g[1], G), dv=oracle.group_reduce(g[2], G), dkv_in=g[-1])
    if token:
        ref["dlog_g"] = g[3]
    for name, r in ref.items():
        emax, efro = harness.rel_errors(got[name], r)
        print(f"  {name:7s} max-rel {emax:.3e} fro-rel {efro:.3e}", flush=True)
        assert np.isfinite(emax) and emax <= TOL["bf16"] and efro <= TOL["bf16"], name


# Two segments, of which the local pass cuts the one it sums in two pieces (local_pieces, from 12 tiles a segment on): the shortest
# that is cut (22 tiles: 12 and 10 of them), the longest that is not (20), pieces of an odd number of 64-token tiles, short last
# tiles, a last segment of a single piece or little more.
@pytest.mark.parametrize("dtype,N", [("bf16", 64 * 24), ("bf16", 64 * 22), ("bf16", 64 * 20), ("bf16", 64 * 25 + 1), ("bf16", 64 * 23 - 37), ("bf16", 64 * 28),
                                     ("f32", 32 * 24), ("f32", 32 * 23 + 7), ("f32", 32 * 28 - 1)])
@pytest.mark.parametrize("D,Dv,token,norm", [(128, 128, False, False), (64, 64, True, False), (64, 128, False, True), (128, 128, True, True)])
def test_local_pass_in_pieces(gpu, oracle, dtype, N, D, Dv, token, norm):
    harness, lasp, si = gpu
    cfg = si.Config("pieces", B=1, H=2, N=N, D=D, chunk=64, dtype=dtype, seed=8700 + N + D, token_decay=token, Dv=Dv)
    inp = si.make_inputs(cfg, with_states=True)
    print(f"case {dtype} N={N} {D}x{Dv} token={token} norm={norm}", flush=True)
    check(harness, oracle, inp, dtype, norm, harness.run_gpu(inp, segments=2, norm_eps=1e-5 if norm else None))


# The same in launches that two sub-sequences share, each in one segment: 86 to 128 heads at d=128 (test_sequence_launches.py has
# the plans), pieces of an even and an odd number of tiles, short last tiles. (The first, a middle and the last head are compared.)
@pytest.mark.parametrize("H,n", PIECES_OF_A_SHARD)
@pytest.mark.parametrize("norm", [False, True])
def test_local_pass_in_pieces_of_a_shard(gpu, oracle, H, n, norm):
    harness, lasp, si = gpu
    cfg = si.Config("pieces", B=1, H=H, N=2 * n, D=128, chunk=64, dtype="bf16", seed=8800 + n)
    inp = si.make_inputs(cfg, with_states=True)
    print(f"case H={H} 2 x {n} norm={norm}", flush=True)
    got = harness.run_gpu(inp, T=2, norm_eps=1e-5 if norm else None)
    heads = [0, H // 2, H - 1]
    few = replace(inp, decay=inp.decay[heads], **{x: np.ascontiguousarray(getattr(inp, x)[:, heads])
                                                  for x in ("q", "k", "v", "dout", "kv_in", "dkv_out")})
    check(harness, oracle, few, "bf16", norm, {x: y[:, heads] for x, y in got.items()})


# 72 heads at d=64, two sub-sequences of three or seven segments: a shared launch that is scanned, or one by one.
@pytest.mark.parametrize("dtype,n", [("bf16", 64 * 12), ("bf16", 64 * 13 - 5), ("f32", 32 * 13 - 3)])
def test_two_sub_sequences_of_several_segments(gpu, oracle, dtype, n):
    harness, lasp, si = gpu
    cfg = si.Config("several", B=1, H=72, N=2 * n, D=64, chunk=64, dtype=dtype, seed=8800 + n)
    inp = si.make_inputs(cfg, with_states=True)
    print(f"case {dtype} 2 x {n}", flush=True)
    check(harness, oracle, inp, dtype, False, harness.run_gpu(inp, T=2))


# bfloat16 d=64 in pairs, cut for two workgroups a CU: 64 heads x 20 tiles, five segments of two pairs; a short last tile; an odd
# last pair (whose cache has a state per tile: by tiles).
@pytest.mark.parametrize("N", [64 * 20, 64 * 20 - 37, 64 * 19])
@pytest.mark.parametrize("token,norm", [(False, False), (True, False), (False, True)])
def test_two_workgroups_a_cu(gpu, oracle, N, token, norm):
    harness, lasp, si = gpu
    cfg = si.Config("two", B=1, H=64, N=N, D=64, chunk=64, dtype="bf16", seed=8900 + N, token_decay=token)
    inp = si.make_inputs(cfg, with_states=True)
    print(f"case N={N} token={token} norm={norm}", flush=True)
    check(harness, oracle, inp, "bf16", norm, harness.run_gpu(inp, norm_eps=1e-5 if norm else None))


def check(harness, oracle, inp, dtype, norm, got):
    decay = None if inp.log_g is not None else inp.decay
    o, kvo = oracle.dims_fwd_brute(inp.q, inp.k, inp.v, decay, inp.kv_in, log_g=inp.log_g)
    dout = inp.dout
    if norm:
        o, rstd = oracle.norm_fwd(o, 1e-5)
        dout = oracle.norm_bwd(inp.dout, o, rstd)
    g = oracle.dims_bwd_brute(inp.q, inp.k, inp.v, dout, decay, inp.kv_in, inp.dkv_out, log_g=inp.log_g)
    ref = dict(out=o, kv_out=kvo, dq=g[0], dk=g[1], dv=g[2], dkv_in=g[-1])
    if inp.log_g is not None:
        ref["dlog_g"] = g[3]
    for name, r in ref.items():
        emax, efro = harness.rel_errors(got[name], r)
        print(f"  {name:7s} max-rel {emax:.3e} fro-rel {efro:.3e}", flush=True)
        assert np.isfinite(emax) and emax <= TOL[dtype] and efro <= TOL[dtype], name
