"""Launch rules that are plain arithmetic (csrc/lasp_rules.h), compiled with the host compiler."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def blocks_for(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", d / "rules.so"
    src.write_text(f'#include "{ROOT}/paper_2404_02882_amd/csrc/lasp_rules.h"\n'
                   'extern "C" void blocks(int ntiles, long long chains, int slots, int *out) {\n'
                   '    const lasp::Blocks b = lasp::blocks_for(ntiles, chains, slots);\n'
                   '    out[0] = b.tiles;\n    out[1] = b.count;\n}\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    fn = ctypes.CDLL(str(lib)).blocks

    def call(ntiles, chains, slots=512):
        out = (ctypes.c_int * 2)()
        fn(ntiles, ctypes.c_longlong(chains), slots, out)
        return out[0], out[1]
    return call


def time_of(tiles, count, chains, slots=512):
    return -(-chains * count // slots) * tiles


def test_bidirectional_blocks(blocks_for):
    """Every tile in exactly one block, and never more rounds x tiles than the share rounded down or up alone gives;
    as long, never fewer workgroups."""
    for chains in (1, 2, 6, 16, 24, 36, 48, 72, 96, 144, 170, 171, 192, 264, 288, 384, 511, 512, 513, 600, 3000):
        for ntiles in (1, 2, 3, 5, 6, 8, 12, 20, 40, 256, 257):
            tiles, count = blocks_for(ntiles, chains)
            assert tiles >= 1 and (count - 1) * tiles < ntiles <= count * tiles
            for want in (512 // chains, -(-512 // chains)):
                t = -(-ntiles // min(max(want, 1), ntiles))
                n = -(-ntiles // t)
                other = time_of(t, n, chains)
                assert time_of(tiles, count, chains) <= other, (chains, ntiles)
                if time_of(tiles, count, chains) == other:
                    assert count >= n, (chains, ntiles)


def test_measured_shapes(blocks_for):
    """Three products of 16 heads x 32768 tokens (128-token tiles) in one round; of 32 heads x 768 tokens in one-tile
    blocks rather than half as many of two; of 128 heads in two blocks each."""
    assert blocks_for(256, 48) == (26, 10)
    assert blocks_for(6, 96) == (1, 6)
    assert blocks_for(20, 384) == (10, 2)
    assert blocks_for(20, 512) == (20, 1)


@pytest.mark.parametrize("dims", [dict(D=128), dict(D=128, kv_heads=1)])
def test_forward_workgroups_stay_within_the_cus(dims):
    """bfloat16 d=128: the automatic forward cut never makes more workgroups than there are CUs while there are no more
    heads than CUs, and uses at least half of them where the sequence has the tiles."""
    from paper_2404_02882_amd import lasp
    for chains in (1, 2, 6, 12, 16, 20, 24, 44, 56, 68, 88, 96, 120, 128, 136, 160, 170, 192, 255, 256):
        for N in (64 * 16, 64 * 64, 64 * 256, 64 * 2048):
            n = lasp.num_segments(lasp.make_shape(1, chains, N, chunk=64, dtype="bf16", **dims))
            assert chains * n <= 256, (chains, N, n)
            # (segments are whole pairs of tiles of one length, so up to half of the share may be lost to rounding)
            assert chains * n >= min(128, chains * (N // 128) // 2), (chains, N, n)


def test_state_cache_of_odd_tile_counts():
    """bfloat16: a state per tile for odd tile counts of short sequences and of d=64, a state per pair otherwise; the
    segments of a short odd sequence are single tiles, whose states the scratch holds."""
    from paper_2404_02882_amd import lasp

    def slots(H, N, D, **kw):
        s = lasp.make_shape(1, H, N, D, 64, "bf16", **kw)
        return lasp.state_cache_bytes(s) / (H * D * (kw.get("Dv") or D) * 2)

    assert [slots(2, N, 128) for N in (448, 447, 385, 384, 512)] == [7, 7, 7, 3, 4]
    assert slots(2, 448, 64, Dv=128) == 7 and slots(16, 64 * 9, 128) == 9      # 144 workgroups
    assert slots(16, 64 * 11, 128) == 6 and slots(32, 5000, 128) == 40
    assert slots(16, 5000, 64) == 79 and slots(16, 5056, 64) == 79 and slots(16, 5120, 64) == 40
    assert slots(2, 448, 128, segments=3) == 7                                 # not a matter of the segments
    assert lasp.scratch_bytes(lasp.make_shape(1, 2, 448, 128, 64, "bf16")) == 2 * 7 * 128 * 128 * 4


def test_short_sequences_scratch():
    """Passes whose workgroups compute their start states themselves use no scratch; the size stays that of the cut they had
    with scanned states (pairs of tiles for even counts), so that buffers of that size still serve."""
    from paper_2404_02882_amd import lasp

    def segments(H, N, D=128, dtype="bf16", **kw):
        s = lasp.make_shape(1, H, N, D, 64, dtype, **kw)
        return lasp.scratch_bytes(s) / (H * D * D * 4)

    assert [segments(2, N) for N in (64, 128, 256, 384, 512, 448, 576, 640)] == [1, 1, 2, 3, 4, 7, 9, 5]
    assert [segments(2, N, 64) for N in (128, 256, 512)] == [1, 2, 4]
    assert [segments(2, N, dtype="f32") for N in (32, 64, 128, 256)] == [1, 2, 4, 8]


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("short")
    src, lib = d / "short.cpp", d / "short.so"
    src.write_text(f'#include "{ROOT}/paper_2404_02882_amd/csrc/lasp_rules.h"\n'
                   'extern "C" int tiles(int want, int ntiles, long long chains, int D, int every, int backward, int alone) {\n'
                   '    return lasp::segment_tiles(want, ntiles, chains, D, every, backward, alone);\n}\n'
                   'extern "C" int own(int tiles, int two_byte) { return lasp::own_states(tiles, two_byte); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    handle = ctypes.CDLL(str(lib))
    handle.tiles.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong] + [ctypes.c_int] * 4
    return handle


def test_short_sequences_alone(rules):
    """Single tiles up to eight of them and a workgroup a CU, whatever the cache holds and only alone; own start states where
    less than eight (float: four) tiles lie in front."""
    assert [rules.own(t, 1) for t in (1, 7, 8)] == [1, 1, 0] and [rules.own(t, 0) for t in (1, 3, 4)] == [1, 1, 0]
    for D in (64, 128):
        for every in (0, 1):
            for backward in (0, 1):
                for ntiles in (1, 2, 7, 8):
                    for want in range(1, ntiles + 1):
                        assert rules.tiles(want, ntiles, 256 // ntiles, D, every, backward, 1) == 1
                        beside = rules.tiles(want, ntiles, 256 // ntiles, D, every, backward, 0)
                        assert rules.tiles(want, ntiles, 256 // ntiles + 1, D, every, backward, 1) == \
                            rules.tiles(want, ntiles, 256 // ntiles + 1, D, every, backward, 0)
                        assert beside >= want and (every or beside % 2 == 0)
                assert rules.tiles(2, 9, 2, D, every, backward, 1) == 2
