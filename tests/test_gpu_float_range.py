"""Float data at the ends of its range: infinities, NaN, the largest finite values and small magnitudes go through the
products as float arithmetic has it. Positive q, k and v, so that every sum an infinity enters is that infinity.
Inside its own 32-token tile a value also meets the zeros of the mask, and 0 x infinity is NaN: rows of the tile in
front of the value are left out."""
from dataclasses import replace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TILE = 32
TOL = 1e-5    # sums of at most 200 positive products in float


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "needs a GPU"
    from paper_2404_02882_amd import harness, synth_inputs
    return harness, synth_inputs


def make(si, N, D, Dv, token, states=True):
    cfg = si.Config("range", B=1, H=2, N=N, D=D, chunk=64, dtype="f32", seed=8400 + N + D + Dv, token_decay=token, Dv=Dv)
    inp = si.make_inputs(cfg, with_states=states)
    pos = lambda x: None if x is None else np.abs(x) + np.float32(1e-3)   # noqa: E731
    return replace(inp, q=pos(inp.q), k=pos(inp.k), v=pos(inp.v), dout=pos(inp.dout), kv_in=pos(inp.kv_in), dkv_out=pos(inp.dkv_out))


def run(harness, oracle, inp, **kw):
    got = harness.run_gpu(inp, **kw)
    with np.errstate(all="ignore"):
        decay = None if inp.log_g is not None else inp.decay
        o, kvo = oracle.dims_fwd_brute(inp.q, inp.k, inp.v, decay, inp.kv_in, log_g=inp.log_g)
        g = oracle.dims_bwd_brute(inp.q, inp.k, inp.v, inp.dout, decay, inp.kv_in, inp.dkv_out, log_g=inp.log_g)
    return got, dict(out=o, kv_out=kvo, dq=g[0], dk=g[1], dv=g[2], dkv_in=g[-1])


def close(name, x, ref):
    """Equal where the reference is not finite, within TOL where it is (all references here are positive)."""
    bad = ~np.isfinite(ref)
    print(f"  {name:7s} non-finite expected {int(bad.sum())}, got {int((~np.isfinite(x)).sum())}", flush=True)
    assert np.array_equal(x[bad], ref[bad], equal_nan=True), name
    assert np.all(np.abs(x[~bad] - ref[~bad]) <= TOL * np.abs(ref[~bad])), name


@pytest.mark.parametrize("D,Dv", [(64, 64), (128, 128), (128, 64)])
@pytest.mark.parametrize("token", [False, True])
@pytest.mark.parametrize("value", [np.inf, np.nan, -np.inf])
def test_non_finite_value(gpu, oracle, D, Dv, token, value):
    """One such v: its column of the state, of every later row of the output and of nothing else."""
    harness, si = gpu
    N, s, c = 200, 71, 13
    inp = make(si, N, D, Dv, token)
    print(f"case {D}x{Dv} token={token} value={value}", flush=True)
    clean, ref = run(harness, oracle, inp, segments=2)
    inp.v[0, 1, s, c] = value
    got, _ = run(harness, oracle, inp, segments=2)
    want = ref["kv_out"].copy()
    want[0, 1, :, c] = value
    close("kv_out", got["kv_out"], want)
    want = ref["out"].copy()
    want[0, 1, s:, c] = value
    rows = np.r_[0:s // TILE * TILE, s:N]
    close("out", got["out"][:, :, rows], want[:, :, rows])
    # gradients that v enters: dq from row s on (every feature), dk of row s
    want = ref["dq"].copy()
    want[0, 1, s:] = value
    close("dq", got["dq"][:, :, rows], want[:, :, rows])
    assert np.array_equal(got["dv"], clean["dv"]) and np.array_equal(got["dkv_in"], clean["dkv_in"])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("big", [np.finfo(np.float32).max, 3.4e38, 2.0 ** 127])
def test_largest_finite_values(gpu, oracle, D, big):
    """A row of k of (near) the largest float against small q, v: finite throughout, and as accurate as anything else."""
    harness, si = gpu
    N, s = 100, 40
    inp = make(si, N, D, D, False, states=False)
    inp.k[0, 0, s] = big
    inp.q *= np.float32(1e-3)
    inp.v *= np.float32(1e-3)
    inp.dout *= np.float32(1e-4)
    print(f"case D={D} big={big}", flush=True)
    got, ref = run(harness, oracle, inp)
    for name in ("out", "kv_out", "dq", "dv", "dk"):
        assert np.isfinite(ref[name]).all()
        close(name, got[name], ref[name])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("scale", [1e-28, 1e-33])
def test_small_magnitudes(gpu, oracle, D, scale):
    """v from 5e-30 (all three bfloat16 parts normal) and from 5e-35 (the last ones subnormal: v to 2^-134, 9e-7 of it)."""
    harness, si = gpu
    inp = make(si, 100, D, D, False, states=False)
    inp = replace(inp, v=(inp.v + np.float32(0.05)) * np.float32(scale))
    print(f"case D={D} scale={scale}", flush=True)
    got, ref = run(harness, oracle, inp)
    for name in ("out", "kv_out", "dq", "dk", "dv", "dkv_in"):
        close(name, got[name], ref[name])


# Forward calls without a cache (up to 256 tokens and 32 heads: k_short; decay 0.5 falls below the smallest float within 256 tokens)
def forward_alone(gpu, oracle, D, lam, N=256):
    harness, si = gpu
    inp = make(si, N, D, D, False)
    if lam is not None:
        inp = replace(inp, decay=np.full_like(inp.decay, lam))
    with np.errstate(all="ignore"):
        o, kvo = oracle.dims_fwd_brute(inp.q, inp.k, inp.v, inp.decay, inp.kv_in)
    return inp, dict(out=o, kv_out=kvo), lambda: harness.run_gpu(inp, backward=False)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("lam", [None, 0.5])
@pytest.mark.parametrize("value", [np.inf, np.nan, -np.inf])
@pytest.mark.parametrize("N,s", [(256, 10), (250, 200)])
def test_non_finite_value_forward_alone(gpu, oracle, D, lam, value, N, s):
    inp, ref, run_it = forward_alone(gpu, oracle, D, lam, N)
    print(f"case forward alone D={D} lambda={lam} value={value} N={N}", flush=True)
    c = 13
    inp.v[0, 1, s, c] = value
    got = run_it()
    ref["kv_out"][0, 1, :, c] = value
    close("kv_out", got["kv_out"], ref["kv_out"])
    ref["out"][0, 1, s:, c] = value
    rows = np.r_[0:s // TILE * TILE, s:N]
    close("out", got["out"][:, :, rows], ref["out"][:, :, rows])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("lam", [None, 0.5])
@pytest.mark.parametrize("N", [100, 230, 256])   # (256: the state's part on a wave that has keys too)
@pytest.mark.parametrize("value", [np.inf, np.nan, -np.inf])
def test_non_finite_state_forward_alone(gpu, oracle, D, lam, N, value):
    inp, ref, run_it = forward_alone(gpu, oracle, D, lam, N)
    print(f"case forward alone, state, D={D} lambda={lam} value={value} N={N}", flush=True)
    inp.kv_in[0, 1, 5, 40] = value
    got = run_it()
    ref["kv_out"][0, 1, 5, 40] = value
    ref["out"][0, 1, :, 40] = value
    for name in ("out", "kv_out"):
        close(name, got[name], ref[name])


@pytest.mark.parametrize("D", [64, 128])
def test_largest_finite_values_forward_alone(gpu, oracle, D):
    inp, _, run_it = forward_alone(gpu, oracle, D, None)
    big = np.finfo(np.float32).max
    inp.k[0, 0, 40] = big
    inp.kv_in[0, 1, 3, 50] = big
    for x in (inp.q, inp.v):
        x *= np.float32(1e-3)
    print(f"case forward alone, largest, D={D}", flush=True)
    o, kvo = oracle.dims_fwd_brute(inp.q, inp.k, inp.v, inp.decay, inp.kv_in)
    assert np.isfinite(o).all() and np.abs(o).max() < big and np.abs(kvo).max() <= big
    got = run_it()
    for name, r in (("out", o), ("kv_out", kvo)):
        close(name, got[name], r)
