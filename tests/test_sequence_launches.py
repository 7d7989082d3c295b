"""What the host layer of a whole sequence (lasp_seq_*, lasp_bidir_seq_*) checks, launches and copies: csrc/lasp*_api.cpp built
with the host compiler against launches that only write down what they were asked for. Addresses are never dereferenced."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2404_02882_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
PIECES_OF_A_SHARD = [(96, 64 * 12), (128, 64 * 12 - 37), (96, 64 * 14), (128, 64 * 13 + 1), (86, 64 * 15 - 5)]   # heads, tokens; bf16, d=128
ERR_NULL, ERR_SHAPE, ERR_WORKSPACE, ERR_ALIAS, ERR_ALIGN = 1, 2, 5, 6, 8

RECORDER = r"""
#include "%(csrc)s/lasp_internal.h"
#include "%(csrc)s/lasp_rules.h"
#include <cstdlib>
#include <cstring>
#include <new>
namespace { int n; long long rec[256][9]; bool no_memory; }
void *operator new(size_t size) {
    if (no_memory) throw std::bad_alloc();
    return std::malloc(size);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
extern "C" void out_of_memory(int yes) { no_memory = yes; }
static hipError_t put(int kind, int shards, const void *a, const void *b, const void *c, const lasp::Plan *p = nullptr) {
    long long r[9] = {kind, shards, (long long)a, (long long)b, (long long)c, p && p->own_states, p ? p->nseg : 0, p ? p->scratch_segs : 0,
                      p ? lasp::local_pieces(p->shards * p->nseg, p->tiles_per_seg, (long long)p->B * p->H) : 0};
    std::memcpy(rec[n++ & 255], r, sizeof r);
    return hipSuccess;
}
extern "C" int recorded(long long *out) {
    std::memcpy(out, rec, sizeof rec);
    const int count = n;
    n = 0;
    return count;
}
namespace lasp {
int tile_tokens(int dtype, int, int) { return dtype == 0 ? 32 : 64; }
hipError_t static_scratch(void **) { return hipErrorUnknown; }
int bidir_reduce_tile(int dtype) { return dtype == 0 ? 32 : 64; }
int bidir_product_tile(int dtype) { return dtype == 0 ? 64 : 128; }
hipError_t launch_bidir_sums(const BidirPlan &, const BidirSums &a, hipStream_t, const KernelEvents *) { return put(4, a.n, a.x[0], a.dq ? a.dq[0] : nullptr, nullptr); }
hipError_t launch_bidir_products(const BidirPlan &, const BidirProducts &a, hipStream_t, const KernelEvents *) { return put(4 + a.nops, a.n, a.x[0][0], a.out[0][0], nullptr); }
hipError_t launch_fwd(const Plan &p, const FwdArgs &a, hipStream_t, const KernelEvents *) {
    return put(a.states_only ? 2 : 0, p.shards, a.k, a.kv_in, a.kv_copy, &p);
}
hipError_t launch_bwd(const Plan &p, const BwdArgs &a, hipStream_t, const KernelEvents *) {
    return put(1, p.shards, a.k, a.dkv_out, a.dkv_copy, &p);
}
hipError_t launch_bidir_apply(const BidirPlan &, const BidirOps &, int, hipStream_t, const KernelEvents *) { return hipErrorUnknown; }
hipError_t launch_bidir_state(const BidirPlan &, const void *, const void *, float *, int, float *, hipStream_t, const KernelEvents *) { return hipErrorUnknown; }
}
extern "C" {
hipError_t hipMemcpyAsync(void *d, const void *s, size_t, hipMemcpyKind, hipStream_t) { return put(3, 0, s, nullptr, d); }
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorUnknown; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorUnknown; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorUnknown; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
}
"""


@pytest.fixture(scope="module")
def api(tmp_path_factory):
    from paper_2404_02882_amd import lasp
    d = tmp_path_factory.mktemp("api")
    src, lib = d / "recorder.cpp", d / "recorder.so"
    src.write_text(RECORDER % dict(csrc=CSRC))
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include",
                    str(src), os.path.join(CSRC, "lasp_api.cpp"), os.path.join(CSRC, "lasp_bidir_api.cpp"), "-o", str(lib)], check=True)
    handle = ctypes.CDLL(str(lib), mode=os.RTLD_LOCAL | os.RTLD_NOW)
    lasp._bind_bidir_sequence(lasp._bind(handle))
    return Api(handle, lasp)


class Sequence:
    """Addresses of a sequence's buffers, all apart unless a test moves one."""

    def __init__(self, T, size=1 << 30):
        self.next = 1 << 40
        self.size = size
        for name in ("q", "k", "v", "out", "rstd", "dout", "log_g", "cache", "dq", "dk", "dv", "dlog_g"):
            setattr(self, name, [self.new() for _ in range(T)])
        self.kv, self.dkv = ([self.new() for _ in range(T + 1)] for _ in range(2))
        self.kv_in, self.dkv_out, self.decay, self.scratch = (self.new() for _ in range(4))

    def new(self):
        self.next += self.size
        return self.next


class Api:
    def __init__(self, lib, lasp):
        self.lib, self.lasp = lib, lasp

    def record(self):
        out = (ctypes.c_longlong * (256 * 9))()
        n = self.lib.recorded(out)
        return [tuple(out[9 * i:9 * i + 9]) for i in range(n)]   # kind (0 forward, 1 backward, 2 states, 3 copy), shards, k, in,
                                                                  # copy, own start states, segments, segments in the scratch,
                                                                  # pieces of a segment in the local pass

    def shape(self, H=4, N=1024, D=64, dtype="bf16", **kw):
        return self.lasp.make_shape(1, H, N, D, 64, dtype, **kw)

    def scratch_bytes(self, shape, T, token=False, recompute=False):
        return self.lib.lasp_seq_scratch_bytes(ctypes.byref(shape), T, int(token), int(recompute))

    @staticmethod
    def table(list_):
        return None if list_ is None else (ctypes.c_size_t * len(list_))(*[x or 0 for x in list_])

    def fwd(self, shape, T, s, token=False, norm=False, cache=True, entering=True, scratch_bytes=None):
        size = self.scratch_bytes(shape, T, token) if scratch_bytes is None else scratch_bytes
        t = self.table
        rc = self.lib.lasp_seq_fwd(ctypes.byref(shape), T, t(s.q), t(s.k), t(s.v), s.kv_in if entering else None,
                                   t(s.log_g if token else [s.decay]), int(token), 1e-5, t(s.out), t(s.rstd) if norm else None,
                                   t(s.kv), t(s.cache) if cache else None, s.scratch, size, None)
        return rc, self.record()

    def bwd(self, shape, T, s, token=False, norm=False, cache=True, entering=True, scratch_bytes=None):
        size = self.scratch_bytes(shape, T, token, not cache) if scratch_bytes is None else scratch_bytes
        t = self.table
        rc = self.lib.lasp_seq_bwd(ctypes.byref(shape), T, t(s.q), t(s.k), t(s.v), t(s.out) if norm else None, t(s.rstd) if norm else None,
                                   t(s.dout), t(s.kv), s.dkv_out if entering else None, t(s.log_g if token else [s.decay]), int(token),
                                   t(s.cache) if cache else None, t(s.dq), t(s.dk), t(s.dv), t(s.dlog_g) if token else None, t(s.dkv),
                                   s.scratch, size, None)
        return rc, self.record()


def groups(records, kinds=(0, 1)):
    return [r[1] for r in records if r[0] in kinds]


@pytest.mark.parametrize("dtype,H,D,N", [("bf16", 4, 64, 1024), ("bf16", 2, 64, 24576), ("bf16", 2, 128, 24576), ("f32", 2, 128, 4096)])
def test_decay_per_token_goes_one_by_one(api, dtype, H, D, N):
    """The gradient of the log decay is a sum over a sub-sequence's tail in which most cancels: every sub-sequence's walk starts
    from the very state (and state gradient) its neighbour's walk returned, and its segments are no longer than alone."""
    shape, T = api.shape(H, N, D, dtype), 4
    s = Sequence(T)
    for cache in (True, False):
        rc, r = api.fwd(shape, T, s, token=True, cache=cache)
        assert rc == 0 and groups(r) == [1] * T
        assert [x[3] for x in r if x[0] == 0] == [s.kv_in] + s.kv[1:T]
        rc, r = api.bwd(shape, T, s, token=True, cache=cache)
        assert rc == 0 and groups(r) == [1] * T
        assert [x[3] for x in r if x[0] == 1] == [s.dkv_out] + s.dkv[T - 1:0:-1]
        rc, r = api.fwd(shape, T, s, cache=cache)   # one lambda per head: together
        assert rc == 0 and groups(r) == [4]
    # and no scratch for several
    one = (api.lib.lasp_gated_scratch_bytes, api.lib.lasp_gated_bwd_recompute_scratch_bytes)
    for recompute, size in enumerate(one):
        assert api.scratch_bytes(shape, T, token=True, recompute=bool(recompute)) == size(ctypes.byref(shape))


def test_caches_are_all_there_or_none(api):
    """A NULL first pointer = no cache; a NULL among the others is refused in both passes before anything is launched (the
    distance to it would send a shared launch to address 0)."""
    T, shape = 4, api.shape()
    for at in (1, 2, 3):
        s = Sequence(T)
        s.cache[at] = None
        assert api.fwd(shape, T, s) == (ERR_NULL, [])
        assert api.bwd(shape, T, s) == (ERR_NULL, [])
    s = Sequence(T)
    s.cache[0] = None   # the others are not looked at
    rc, r = api.fwd(shape, T, s)
    assert rc == 0 and groups(r) == [4]
    rc, r = api.bwd(shape, T, s)   # states rebuilt: more scratch
    assert (rc, r) == (ERR_WORKSPACE, [])
    rc, r = api.bwd(shape, T, s, scratch_bytes=api.scratch_bytes(shape, T, recompute=True))
    assert rc == 0 and groups(r, (1, 2)) == [4, 4]


def test_states_between_are_needed_where_they_are_rebuilt(api):
    """Only the state in front of the first sub-sequence may be absent (zeros)."""
    T, shape = 3, api.shape(segments=1)
    s = Sequence(T)
    s.kv[0] = None
    assert api.bwd(shape, T, s, cache=False)[0] == 0 and api.bwd(shape, T, s)[0] == 0
    s.kv[1] = None
    assert api.bwd(shape, T, s, cache=False) == (ERR_NULL, [])
    assert api.bwd(shape, T, s)[0] == 0   # with caches they are not read


def test_copy_of_the_entering_state_among_other_sub_sequences_buffers(api):
    """kv[0] (dkv[T]) is written by the first (last) sub-sequence's walk. On what another one reads it is refused, on what
    another one writes the sequence goes one by one, in whose order the later write stays; the other groups stay together."""
    T, shape = 6, api.shape()
    for buf in ("q", "k", "v"):
        for t in range(T):
            s = Sequence(T)
            s.kv[0] = getattr(s, buf)[t]
            assert api.fwd(shape, T, s) == (ERR_ALIAS, []), (buf, t)
            assert api.fwd(shape, T, s, entering=False)[0] == 0   # not written then
    s = Sequence(T)
    s.kv[0] = s.decay
    assert api.fwd(shape, T, s) == (ERR_ALIAS, [])
    for buf in ("q", "k", "v", "dout", "cache", "out", "rstd"):
        for t in range(T):
            s = Sequence(T)
            s.dkv[T] = getattr(s, buf)[t]
            assert api.bwd(shape, T, s, norm=True) == (ERR_ALIAS, []), (buf, t)
    s = Sequence(T)
    s.dkv[T] = s.kv[0]   # read where the states are rebuilt
    assert api.bwd(shape, T, s, cache=False) == (ERR_ALIAS, [])
    assert api.bwd(shape, T, s)[0] == 0
    group = 3
    assert groups(api.fwd(shape, T, Sequence(T))[1]) == [group] * 2 == groups(api.bwd(shape, T, Sequence(T))[1])
    for buf, t in [("out", 1), ("out", 2), ("cache", 1), ("rstd", 2), ("kv", 2), ("kv", 3)]:   # kv[0] = kv[2]: states in turn
        s = Sequence(T)
        s.kv[0] = getattr(s, buf)[t]
        rc, r = api.fwd(shape, T, s, norm=True)
        assert rc == 0 and groups(r) == [1, 1, 1, 3], (buf, t)
        assert [x[4] for x in r] == [s.kv[0], 0, 0, 0]
    for buf, t in [("dq", 4), ("dk", 3), ("dv", 4), ("dkv", 4), ("dkv", 3)]:
        s = Sequence(T)
        s.dkv[T] = getattr(s, buf)[t]
        rc, r = api.bwd(shape, T, s)
        assert rc == 0 and groups(r) == [1, 1, 1, 3], (buf, t)
        assert [x[4] for x in r] == [s.dkv[T], 0, 0, 0]
    s = Sequence(T)
    s.kv[0] = s.out[4]   # a group after the one that writes it
    assert groups(api.fwd(shape, T, s)[1]) == [3, 3]


def test_refused_calls_copy_nothing(api):
    """An entering state that lies in what the call writes is copied first, but only by a call that passes its checks; a state
    that overlaps its own copy in part is refused."""
    T, shape = 3, api.shape()
    state = 4 * 64 * 64 * 4
    for copied, place in (("fwd", lambda s: setattr(s, "kv_in", s.kv[T])), ("bwd", lambda s: setattr(s, "dkv_out", s.dkv[0])),
                          ("fwd", lambda s: setattr(s, "kv_in", s.kv_in + 4)), ("bwd", lambda s: setattr(s, "dkv_out", s.dkv_out + 4))):
        s = Sequence(T)
        place(s)
        src, dst = (s.kv_in, s.kv[0]) if copied == "fwd" else (s.dkv_out, s.dkv[T])
        rc, r = getattr(api, copied)(shape, T, s)
        assert rc == 0 and r[0][0] == 3 and (r[0][2], r[0][4]) == (src, dst)
        assert r[1][3] == dst and groups(r) == [3] and [x[4] for x in r[1:]] == [0]
        s.q[2] += 8
        assert getattr(api, copied)(shape, T, s) == (ERR_ALIGN, [])
        s.q[2] = s.out[2] if copied == "fwd" else s.dq[2]
        assert getattr(api, copied)(shape, T, s) == (ERR_ALIAS, [])
    for call in (api.fwd, api.bwd):   # nor onto what another sub-sequence reads
        s = Sequence(T)
        s.kv_in, s.dkv_out, s.kv[0], s.dkv[T] = s.kv_in + 4, s.dkv_out + 4, s.q[1], s.q[1]
        assert call(shape, T, s) == (ERR_ALIAS, [])
    for off in (16, state - 16, -16):
        s = Sequence(T)
        s.kv[0], s.dkv[T] = s.kv_in + off, s.dkv_out + off
        assert api.fwd(shape, T, s) == (ERR_ALIAS, []) == api.bwd(shape, T, s)
    s = Sequence(T)
    s.kv[0], s.dkv[T] = s.kv_in, s.dkv_out   # in place already
    for call in (api.fwd, api.bwd):
        rc, r = call(shape, T, s)
        assert rc == 0 and groups(r) == [3] and [x[0] for x in r].count(3) == 0 and r[0][4] == 0


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D", [64, 128])
def test_segments_fit_the_scratch(api, dtype, D):
    """Every pass that goes through its segments' states in the scratch finds room for them there."""
    for H in (1, 2, 16, 32, 86, 128, 300):
        for N in (1, 64, 65, 128, 191, 192, 256, 448, 500, 512, 513, 640, 1000, 5000):
            for token in (False, True):
                for T in (1, 3):
                    shape, s = api.shape(H, N, D, dtype), Sequence(T)
                    records = api.fwd(shape, T, s, token)[1] + api.bwd(shape, T, s, token)[1] + api.bwd(shape, T, s, token, cache=False)[1]
                    assert len(records) >= 3
                    for r in records:
                        assert r[5] or r[6] <= r[7], (H, N, token, T, r)
                        assert not r[5] or r[1] == 1


def test_parts_of_grouped_heads_stay_bounded(api):
    """Grouped K/V heads: dK, dV parts of every sub-sequence of a launch lie in the scratch at once, up to 1 GiB."""
    T, H = 4, 16
    for N, sizes in ((4096, [4]), (32768, [4]), (32832, [2, 2]), (65536, [2, 2]), (65600, [1] * 4), (262144, [1] * 4)):
        shape = api.shape(H, N, 128, kv_heads=4)
        rc, r = api.bwd(shape, T, Sequence(T))
        assert rc == 0 and groups(r) == sizes, N
        one = api.lib.lasp_scratch_bytes(ctypes.byref(shape))
        assert api.scratch_bytes(shape, T) <= one + (1 << 30)
        if len(sizes) == T:
            assert api.scratch_bytes(shape, T) == one
    plain = api.shape(H, 65536, 128)
    assert groups(api.bwd(plain, T, Sequence(T))[1]) == [4]   # no parts


def test_groups_of_about_one_size_and_what_is_left_over(api):
    """(The sequences that the GPU tests of shared launches take as ragged, over several tiles, or with one left over.)"""
    for H, dtype, D, Dv, n, T, sizes in ((32, "bf16", 128, 0, 1050, 2, [2]), (32, "bf16", 128, 64, 1180, 2, [2]), (32, "f32", 128, 0, 1000, 2, [2]),
                                         (4, "bf16", 128, 0, 130, 13, [4, 4, 4, 1]), (4, "f32", 64, 0, 40, 13, [4, 4, 4, 1]),
                                         (100, "bf16", 64, 0, 130, 3, [2, 1]), (4, "bf16", 64, 0, 64, 9, [3, 3, 3]), (257, "bf16", 64, 0, 64, 4, [1] * 4)):
        shape, s = api.shape(H, n, D, dtype, Dv=Dv), Sequence(T)
        rc, r = api.fwd(shape, T, s)
        assert rc == 0 and groups(r) == sizes
        if sizes == [2]:   # ragged last segments of several tiles of the local pass
            tile, local = (32, 32) if dtype == "f32" else (64, 64 if Dv else 128)
            tiles = -(-n // tile)
            per_seg = -(-tiles // r[0][6])
            per_seg += per_seg % 2 if dtype == "bf16" else 0
            last = n - (r[0][6] - 1) * per_seg * tile
            assert last % local and last > local, (H, dtype, last)
        rc, r = api.bwd(shape, T, s)
        assert rc == 0 and groups(r) == sizes[::-1]
        assert [x[5] for x in r if x[1] > 1] == [0] * sum(g > 1 for g in sizes)   # start states from the scratch


def test_rejects_before_launch(api):
    T, shape = 3, api.shape()
    lib, by = api.lib, ctypes.byref
    assert api.scratch_bytes(shape, 0) == api.scratch_bytes(shape, -1) == api.scratch_bytes(api.shape(D=96), T) == 0
    assert api.scratch_bytes(shape, 1) == lib.lasp_scratch_bytes(by(shape))
    for token in (False, True):
        for norm in (False, True):
            need = {"fwd": ["q", "k", "v", "out"], "bwd": ["q", "k", "v", "dout", "dq", "dk", "dv"]}
            need["fwd"] += ["log_g"] * token + ["rstd"] * norm
            need["bwd"] += ["log_g", "dlog_g"] * token + ["out", "rstd"] * norm
            for name, call in (("fwd", api.fwd), ("bwd", api.bwd)):
                assert call(shape, T, Sequence(T), token, norm)[0] == 0
                for buf in need[name]:
                    for t in range(T):
                        s = Sequence(T)
                        getattr(s, buf)[t] = None
                        assert call(shape, T, s, token, norm) == (ERR_NULL, []), (name, buf, t)
                        s = Sequence(T)
                        getattr(s, buf)[t] += 4
                        assert call(shape, T, s, token, norm) == (ERR_ALIGN, []), (name, buf, t)
                size = api.scratch_bytes(shape, T, token)
                assert call(shape, T, Sequence(T), token, norm, scratch_bytes=size - 1) == (ERR_WORKSPACE, [])
                for bad in (0, -2):
                    s = Sequence(T)
                    assert (lib.lasp_seq_fwd(by(shape), bad, *[api.table(x) for x in (s.q, s.k, s.v)], s.kv_in, api.table([s.decay]), 0, 0.0, api.table(s.out),
                                             None, api.table(s.kv), None, s.scratch, size, None) == ERR_SHAPE)
                for t in range(T):
                    s = Sequence(T)
                    (s.out if name == "fwd" else s.dq)[t] = s.q[t]
                    assert call(shape, T, s, token, norm) == (ERR_ALIAS, [])
                    s = Sequence(T)
                    (s.kv if name == "fwd" else s.dkv)[t + (name == "fwd")] = s.scratch
                    assert call(shape, T, s, token, norm) == (ERR_ALIAS, [])
    recompute = api.scratch_bytes(shape, T, recompute=True)
    assert api.bwd(shape, T, Sequence(T), cache=False, scratch_bytes=recompute - 1) == (ERR_WORKSPACE, [])
    s = Sequence(T)   # whole lists
    args = [by(shape), T, *[api.table(x) for x in (s.q, s.k, s.v)], s.kv_in, api.table([s.decay]), 0, 0.0, api.table(s.out), None,
            api.table(s.kv), None, s.scratch, recompute, None]
    for at in (2, 3, 4, 6, 9, 11):
        assert lib.lasp_seq_fwd(*args[:at], None, *args[at + 1:]) == ERR_NULL
    args = [by(shape), T, *[api.table(x) for x in (s.q, s.k, s.v)], None, None, api.table(s.dout), api.table(s.kv), s.dkv_out,
            api.table([s.decay]), 0, None, *[api.table(x) for x in (s.dq, s.dk, s.dv)], None, api.table(s.dkv), s.scratch, recompute, None]
    for at in (2, 3, 4, 7, 8, 10, 13, 14, 15, 17):
        assert lib.lasp_seq_bwd(*args[:at], None, *args[at + 1:]) == ERR_NULL
    assert api.record() == []


def test_local_pass_of_two_sub_sequences_in_pieces(api):
    """(The sequences that the GPU test of pieces in shared launches takes: one segment each, two pieces of it, in both passes.)"""
    for H, n in PIECES_OF_A_SHARD:
        shape, s = api.shape(H, n, 128), Sequence(2)
        for cache in (True, False):
            for rc, r in (api.fwd(shape, 2, s, cache=cache), api.bwd(shape, 2, s, cache=cache, norm=True)):
                assert rc == 0 and len(r) in (1, 2) and all((x[1], x[6], x[8]) == (2, 1, 2) for x in r), (H, n, r)


# Bidirectional sequences whose dQ comes with the sum: dtype, d, heads, lengths (the GPU test takes them, too)
DQ_WITH_SUM = [("bf16", 64, 64, [192, 200]), ("bf16", 128, 64, [200, 129, 1]), ("f32", 64, 64, [100, 97]), ("f32", 128, 64, [200, 40, 5, 1])]


def bidir(api, dtype, D, H, lengths, moved=()):
    """Records of the forward and of the backward call: (4 sum / 4 + number of products, sub-sequences, first input, first output)."""
    T, s = len(lengths), Sequence(len(lengths))
    for a, i, b, j in moved:
        getattr(s, a)[i] = getattr(s, b)[j]
    shapes = (api.lasp.Shape * T)(*[api.shape(H, n, D, dtype) for n in lengths])
    size = api.lib.lasp_bidir_seq_scratch_bytes(shapes, T)
    t = api.table
    fwd = api.lib.lasp_bidir_seq_fwd(shapes, T, t(s.q), t(s.k), t(s.v), s.kv_in, t(s.out), s.scratch, size, None), api.record()
    bwd = api.lib.lasp_bidir_seq_bwd(shapes, T, t(s.q), t(s.k), t(s.v), t(s.dout), s.kv_in, s.dkv_out, t(s.dq), t(s.dk), t(s.dv), s.scratch,
                                     size, None), api.record()
    return s, fwd, bwd


def test_bidirectional_launches(api):
    """Up to four sub-sequences a launch; dQ with the sum where that fills the device and is long enough to pay, with the other
    products elsewhere; an output over another sub-sequence's input: one by one, dQ behind the sum."""
    for dtype, D, H, lengths in DQ_WITH_SUM:
        s, (rc, f), (rc2, b) = bidir(api, dtype, D, H, lengths)
        n = len(lengths)
        assert rc == rc2 == 0 and [x[:4] for x in f] == [(4, n, s.k[0], 0), (5, n, s.q[0], s.out[0])]
        assert [x[:4] for x in b] == [(4, n, s.q[0], s.dq[0]), (6, n, s.v[0], s.dk[0])], (dtype, D)
    apart = [("bf16", 128, 16, [1152]), ("bf16", 128, 32, [636]), ("bf16", 128, 2, [8192]), ("bf16", 128, 3, [16512]), ("bf16", 64, 128, [768]),
             ("bf16", 64, 3, [64, 1, 127, 200]), ("f32", 64, 128, [1024]), ("f32", 64, 2, [21705]), ("f32", 64, 32, [384])]
    for dtype, D, H, lengths in apart:
        s, _, (rc, b) = bidir(api, dtype, D, H, lengths)
        assert rc == 0 and [x[:4] for x in b] == [(4, len(lengths), s.q[0], 0), (7, len(lengths), s.dout[0], s.dq[0])], (dtype, D, H)
    s, (rc, f), (rc2, b) = bidir(api, "bf16", 64, 64, [192] * 5)
    assert rc == rc2 == 0 and [x[:2] for x in f] == [(4, 4), (4, 1), (5, 4), (5, 1)] and [x[:2] for x in b] == [(4, 4), (4, 1), (6, 4), (6, 1)]
    for moved in (("dq", 0, "q", 0), ("dk", 1, "k", 0), ("dv", 0, "dout", 1)):
        s, _, (rc, b) = bidir(api, "bf16", 64, 64, [192, 192], [moved])
        assert rc == 0 and [x[:2] for x in b] == [(4, 2), (7, 1), (7, 1)] and b[0][3] == 0, moved
    s, (rc, f), _ = bidir(api, "bf16", 64, 64, [192, 192], [("out", 0, "q", 1)])
    assert rc == 0 and [x[:2] for x in f] == [(4, 2), (5, 1), (5, 1)]


def test_host_memory_runs_out(api):
    """What the buffers are compared in cannot be had: one sub-sequence after the other, which needs no comparison."""
    shape, T, s = api.shape(), 3, Sequence(3)
    api.lib.out_of_memory(1)
    try:
        (rc, f), (rc2, b), (_, (rc3, bf), (rc4, bb)) = api.fwd(shape, T, s), api.bwd(shape, T, s), bidir(api, "bf16", 64, 64, [192, 192])
    finally:
        api.lib.out_of_memory(0)
    assert rc == rc2 == rc3 == rc4 == 0 and groups(f) == groups(b) == [1] * T
    assert [x[:2] for x in bf] == [(4, 2), (5, 1), (5, 1)] and [x[:2] for x in bb] == [(4, 2), (7, 1), (7, 1)]
