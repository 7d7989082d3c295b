"""bfloat16 forward walks of d_k = d_v = 128 on both sides of 256 workgroups (eight waves a workgroup up to there,
four from 257 on), with and without a cache (states rebuilt), whole and ragged lengths, both decay models, Norm,
against the fp64 oracle. Outputs and inputs are rounded once to bfloat16: 2e-2 as everywhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-2
EPS = 1e-5


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "needs a GPU"
    from paper_2404_02882_amd import harness, synth_inputs
    return harness, synth_inputs


@pytest.mark.parametrize("H", [64, 65])   # one segment each: 256 and 260 workgroups
@pytest.mark.parametrize("N", [128, 97])
@pytest.mark.parametrize("token", [False, True])
@pytest.mark.parametrize("norm,recompute", [(False, False), (True, False), (False, True)])
def test_both_sides(gpu, oracle, H, N, token, norm, recompute):
    harness, si = gpu
    cfg = si.Config("waves", B=4, H=H, N=N, D=128, chunk=64, dtype="bf16", seed=5300 + N + H, token_decay=token)
    print(f"case H={H} N={N} token={token} norm={norm} recompute={recompute}", flush=True)
    inp = si.make_inputs(cfg, with_states=True)
    got = harness.run_gpu(inp, norm_eps=EPS if norm else None, recompute=recompute)
    if token:
        o, kvo = oracle.gated_fwd_brute(inp.q, inp.k, inp.v, inp.log_g, inp.kv_in)
    else:
        o, kvo = oracle.fwd_brute(inp.q, inp.k, inp.v, inp.decay, inp.kv_in)
    dout, y = inp.dout, o
    if norm:
        y, rstd = oracle.norm_fwd(o, EPS)
        dout = oracle.norm_bwd(inp.dout, y, rstd)
    if token:
        dq, dk, dv, _, gin = oracle.gated_bwd_brute(inp.q, inp.k, inp.v, dout, inp.log_g, inp.kv_in, inp.dkv_out)
    else:
        dq, dk, dv, gin = oracle.bwd_brute(inp.q, inp.k, inp.v, dout, inp.decay, inp.kv_in, inp.dkv_out)
    for name, r in dict(out=y, kv_out=kvo, dq=dq, dk=dk, dv=dv, dkv_in=gin).items():
        emax, efro = harness.rel_errors(got[name], r)
        print(f"  {name:7s} max-rel {emax:.3e} fro-rel {efro:.3e}", flush=True)
        assert np.isfinite(emax) and emax <= TOL and efro <= TOL, name
