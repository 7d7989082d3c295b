"""GPU parity of forward calls of a few tokens that keep no state cache (one kernel runs the token recurrence up
to 12 tokens, the tile walk from 13 on) against the fp64 oracle: around that length, both data types, both decay
models, key and value dimensions 64 and 128, grouped heads, with and without an entering state, chained.
float: at most 128 products and 12 decays a sum, so 1e-5; bfloat16: outputs rounded once, 2e-2 as everywhere."""
from dataclasses import replace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "needs a GPU"
    from paper_2404_02882_amd import harness, synth_inputs
    return harness, synth_inputs


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("token", [False, True])
@pytest.mark.parametrize("N,T,D,Dv,G,states", [(1, 1, 128, 128, 1, True), (2, 1, 64, 64, 1, False), (11, 1, 64, 128, 2, True),
                                               (12, 1, 128, 64, 1, True), (13, 1, 128, 128, 4, True), (36, 3, 128, 128, 2, True)])
def test_few_tokens(gpu, oracle, dtype, token, N, T, D, Dv, G, states):
    harness, si = gpu
    cfg = si.Config("step", B=2, H=4, N=N, D=D, chunk=64, dtype=dtype, T=T, seed=5200 + N, token_decay=token, Dv=Dv)
    inp = si.make_inputs(cfg, with_states=states)
    inp = replace(inp, k=inp.k[:, ::G].copy(), v=inp.v[:, ::G].copy())
    k, v = oracle.group_expand(inp.k, G), oracle.group_expand(inp.v, G)
    ref = oracle.dims_fwd_brute(inp.q, k, v, None if token else inp.decay, inp.kv_in, log_g=inp.log_g)
    got = harness.run_gpu(inp, T=T, backward=False)
    for name, r in zip(("out", "kv_out"), ref):
        emax, efro = harness.rel_errors(got[name], r)
        print(f"  {dtype} N{N} T{T} {D}x{Dv} G{G} {name}: max-rel {emax:.3e} fro-rel {efro:.3e}", flush=True)
        assert got[name].shape == r.shape and np.isfinite(emax) and emax <= TOL[dtype] and efro <= TOL[dtype], name
