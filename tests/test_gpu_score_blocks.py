"""Float data: the score tile of 32 tokens goes through the matrix cores as 16x16 blocks, the one above the diagonal is
never computed. Lengths around the blocks' edges against the brute-force oracle (1e-5: sums of at most 128 products with
errors of 2^-24 each), and outputs of earlier tokens that do not change with what later tokens hold."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("token", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N", [13, 16, 17, 31, 33, 48])
def test_block_edges(oracle, N, D, token):
    from paper_2404_02882_amd import harness
    from paper_2404_02882_amd import synth_inputs as si
    print(f"case score blocks N={N} D={D} token={token}", flush=True)
    inp = si.make_inputs(si.Config("blocks", B=1, H=2, N=N, D=D, chunk=64, dtype="f32", seed=N + D, token_decay=token), with_states=True)
    if token:
        inp.log_g = np.log(np.random.default_rng(N).uniform(0.8, 1.0, (1, 2, N))).astype(np.float32)
    else:
        inp.decay = np.array([0.8, 1.0], dtype=np.float32)
    got = harness.run_gpu(inp)
    if token:
        o, kvo = oracle.gated_fwd_brute(inp.q, inp.k, inp.v, inp.log_g, inp.kv_in)
        dq, dk, dv, _, gin = oracle.gated_bwd_brute(inp.q, inp.k, inp.v, inp.dout, inp.log_g, inp.kv_in, inp.dkv_out)
    else:
        o, kvo = oracle.fwd_brute(inp.q, inp.k, inp.v, inp.decay, inp.kv_in)
        dq, dk, dv, gin = oracle.bwd_brute(inp.q, inp.k, inp.v, inp.dout, inp.decay, inp.kv_in, inp.dkv_out)
    for name, r in dict(out=o, kv_out=kvo, dq=dq, dk=dk, dv=dv, dkv_in=gin).items():
        emax, efro = harness.rel_errors(got[name], r)
        assert np.isfinite(emax) and emax <= 1e-5 and efro <= 1e-5, (name, emax, efro)
    # later tokens replaced: what comes before them stays as it is
    at = min(N - 1, 16)
    for x in (inp.k, inp.v, inp.q, inp.dout):
        x[:, :, at:] *= -3.0
    again = harness.run_gpu(inp)
    assert np.array_equal(got["out"][:, :, :at], again["out"][:, :, :at])
