// C-ABI host layer: argument validation, launch planning, dispatch. No device
// memory is allocated or freed here and nothing synchronises; see include/lasp.h.
#include "../../include/lasp.h"
#include "../../include/lasp_profile.h"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <utility>
#include <vector>

#include "lasp_checks.h"
#include "lasp_internal.h"
#include "lasp_rules.h"

namespace {

using lasp::check_buffers;
using lasp::elem_bytes;
using lasp::next_slot;
using lasp::overlap;
using lasp::overlap_any;
using lasp::Span;
using lasp::Together;

// Segments per head when the caller leaves the choice to the library: about as many workgroups (B*H*segments) as
// the device has CUs, never more than one segment per tile. A second forward workgroup per CU (512) hides more
// latency but doubles the segment states that go through memory: bf16 d=128 forward, 512 against 256 workgroups,
// 16 heads x 32768 tokens 208 / 197 us, 32 x 4096 69 / 65, 256 x 4096 (two segments / one, no local pass) 345 / 285.
// Never more workgroups than CUs where it can be helped: a few left over are a whole second round (backward, 12 heads x
// 32768: 22 segments 348 us, 20 segments 235), and the forward walk in eight waves takes a CU to itself (forward, the
// nearest count / rounded down: 24 heads x 16384 tokens 264 / 240 workgroups 200 / 152 us, 56 x 4096 111 / 86,
// 136 x 16384 950 / 805 with 272 / 136).
// With a key or value dimension of 64 a state is a quarter or half of the bytes and a tile brings less to stream,
// so 512 forward workgroups win, and two share a CU, so the count may be the nearest: 16 x 32768 at d=64 87 / 107 us;
// d_k=64, d_v=128 norm step of 32 x 5504, two shards, 352 / 376.
// Float walks are bound by vector and matrix instructions issued one after the
// other, which a second workgroup per CU overlaps: 512 (16 x 8192 at d=128 forward 157 / 148 us), except the 8-wave
// backward walk at d=128, of which one fits (per-token decay 386 / 409 us).
constexpr int kTargetWorkgroups = lasp::kOnePerCu;
constexpr int kTargetWorkgroupsLatencyBound = 2 * lasp::kOnePerCu;
enum Pass { kForward = 0, kBackward = 1 };

bool valid_dims(const lasp_shape *s) {
    if (!s) return false;
    if (s->B <= 0 || s->H <= 0 || s->N <= 0) return false;
    if (s->D != 64 && s->D != 128) return false;
    if (s->chunk != 64 && s->chunk != 128 && s->chunk != 256) return false;
    if ((int64_t)s->B * s->H > 65535) return false;  // grid.y limit
    if (s->kv_heads < 0 || (s->kv_heads > 0 && (s->kv_heads > s->H || s->H % s->kv_heads != 0))) return false;
    if (s->Dv != 0 && s->Dv != 64 && s->Dv != 128) return false;
    return true;
}

// Segments per head of a pass when the caller leaves the choice to the library. chains: heads times the sub-sequences that
// go through one launch.
int auto_segments(const lasp::Plan &p, Pass pass, int64_t chains) {
    const bool two_per_cu = p.dtype == LASP_F32 ? pass == kForward || p.D == 64 : pass == kForward && (p.dk == 64 || p.dv == 64);
    const int target = two_per_cu ? kTargetWorkgroupsLatencyBound : kTargetWorkgroups;
    int64_t round = two_per_cu && pass == kForward ? chains / 2 : 0;
    // Three workgroups of the d=64 forward walk fit a CU. With a decay per token, which keeps them longer at the tables, the
    // count is rounded up: 100 heads x 8000 tokens, five / six segments 152 / 142 us.
    if (p.dtype == LASP_BF16 && p.D == 64 && p.token && pass == kForward) round = chains - 1;
    int want = (int)((target + round) / chains);
    // Backward at d=64, two workgroups a CU. By tiles: 48 heads x 5056 tokens, 5 / 6 / 10 segments 79 / 90 / 67 us,
    // 100 x 5056, 2 / 3 / 5 174 / 169 / 140; past 32 segments the scan costs more (8 x 5056, 32 / 64 28.3 / 31.1). In pairs, from two pairs a segment
    // on, one / two workgroups a CU: 16 heads x 32768 tokens 258 / 240 us, 32 x 4096 86.3 / 82.0, 128 x 1024 78.8 / 72.9, but (one pair a
    // segment) 16 x 4 x 1024 in shared launches 62.1 / 62.8, and 128 segments of few heads stay (2 x 32768, 32 / 128 133 / 95).
    if (p.dtype == LASP_BF16 && p.D == 64 && pass == kBackward) {
        const int two = (int)std::min<int64_t>(kTargetWorkgroupsLatencyBound / chains, 32);
        want = p.cache_tiles == 1 ? two : std::max(want, std::min(two, p.ntiles / 4));
    }
    if (want > p.ntiles) want = p.ntiles;
    return want < 1 ? 1 : want;
}

bool two_byte_dtype(const lasp_shape *s) { return s->dtype == LASP_BF16; }

// group: sub-sequences that a launch takes (at most)
int make_plan(const lasp_shape *s, Pass pass, lasp::Plan *p, bool token = false, bool norm = false, int group = 1) {
    if (!s) return LASP_ERR_NULL;
    if (s->dtype != LASP_F32 && s->dtype != LASP_BF16) return LASP_ERR_DTYPE;
    if (!valid_dims(s)) return LASP_ERR_SHAPE;
    p->B = s->B;
    p->H = s->H;
    p->N = s->N;
    p->dk = s->D;
    p->dv = s->Dv != 0 ? s->Dv : s->D;
    p->D = p->dk > p->dv ? p->dk : p->dv;   // the kernels' dimension; the narrower of the two is zero-padded on chip
    p->dtype = s->dtype;
    p->kvdiv = s->kv_heads > 0 ? s->H / s->kv_heads : 1;
    p->tile = lasp::tile_tokens(s->dtype, s->chunk, p->D);
    p->ntiles = (s->N + p->tile - 1) / p->tile;
    int want = s->segments;
    if (want < 0 || want > p->ntiles) return LASP_ERR_SHAPE;
    const bool two_byte = two_byte_dtype(s);   // tiles are walked in pairs, or one by one
    // Float segments are no longer than a launch of one sub-sequence cuts them: a sum's rounding error grows with the length of
    // the chain it is built in (32 heads x 1024 x 4, d=128: 3.9e-7 with a quarter of the segments, 3.2e-7 so).
    const int64_t chains = (int64_t)s->B * s->H * (two_byte_dtype(s) ? group : 1);
    p->shards = 1;
    p->token = token;
    p->norm = norm;
    if (two_byte) {   // (whatever the group: the layout of a sub-sequence's cache does not depend on the others)
        p->cache_tiles = lasp::cache_every_tile(p->ntiles, (int64_t)s->B * s->H, p->D) ? 1 : 2;
    } else {
        const int fwd_auto = auto_segments(*p, kForward, chains);
        p->cache_tiles = (p->ntiles + fwd_auto - 1) / fwd_auto;
    }
    if (want == 0) want = auto_segments(*p, pass, chains);
    const bool alone = s->segments == 0 && group == 1;   // a launch of one sub-sequence, cut as the library likes
    p->ragged = s->N % (two_byte && pass == kBackward ? 2 * p->tile : p->tile) != 0;
    auto segments = [&](int tiles) { return (p->ntiles + tiles - 1) / tiles; };   // every segment non-empty
    const int share = segments(want);
    auto tiles = [&](bool single) {
        return two_byte ? lasp::segment_tiles(share, p->ntiles, chains, p->D, p->cache_tiles == 1, pass == kBackward, single) : share;
    };
    p->tiles_per_seg = tiles(alone);
    p->nseg = segments(p->tiles_per_seg);
    // (the backward walk in pairs has no room for it: with it in, its loop comes out 2 - 4 % slower)
    p->own_states = alone && p->nseg > 1 && lasp::own_states((p->nseg - 1) * p->tiles_per_seg, two_byte) &&
                    (!two_byte || pass == kForward || p->tiles_per_seg == 1 || p->cache_tiles == 1);
    // The scratch is that of the cut without the rule for short sequences that go through alone: where that makes more
    // segments, the workgroups compute their own start states and no scratch is touched.
    p->scratch_segs = segments(tiles(false));
    return LASP_OK;
}

size_t cache_bytes(const lasp_shape *shape, bool token) {
    lasp::Plan p;
    if (make_plan(shape, kForward, &p, token) != LASP_OK) return 0;
    return (size_t)p.B * p.H * ((p.ntiles + p.cache_tiles - 1) / p.cache_tiles) * p.dk * p.dv * elem_bytes(p.dtype);   // [d_k][d_v] per slot
}

// Scratch layout: [segment states][per-token decay only: segment log-decays][.. : per-token r_t]
// [one lambda per head and a short last tile only: unused, keeps the size callers have been told]
// [grouped K/V heads only: dK, dV per query head].
struct ScratchLayout {
    size_t states, seglog, rtok, dk_part, dv_part, total;  // byte offsets of the regions (states = 0), total size
};
size_t round256(size_t x) { return (x + 255) / 256 * 256; }
bool scratch_layout(const lasp_shape *shape, bool token, ScratchLayout *l, int group = 1) {
    lasp::Plan f, b;
    const size_t chains = (size_t)(shape ? shape->B : 0) * (shape ? shape->H : 0);
    size_t nseg = 0;   // of all sub-sequences of a launch; one buffer serves both passes, and launches of one sub-sequence
    for (int n = group; n >= 1; n = n > 1 ? 1 : 0) {
        if (make_plan(shape, kForward, &f, token, false, n) != LASP_OK || make_plan(shape, kBackward, &b, token, false, n) != LASP_OK)
            return false;
        nseg = std::max<size_t>(nseg, n * std::max(f.scratch_segs, b.scratch_segs));
    }
    l->states = 0;
    l->seglog = round256(chains * nseg * f.dk * f.dv * sizeof(float));   // segment states, [d_k][d_v] floats each
    l->rtok = l->seglog;
    size_t end = l->seglog;
    const bool ragged = f.N % f.tile != 0;
    if (f.token || ragged) {
        const size_t per_token = round256(chains * (size_t)f.N * sizeof(float));
        l->rtok = l->seglog + round256(chains * nseg * sizeof(float));
        end = l->rtok + (f.token ? 1 : 2) * per_token;
    }
    l->dk_part = l->dv_part = end;
    if (f.kvdiv > 1) {
        l->dv_part = l->dk_part + round256(group * chains * f.N * f.dk * elem_bytes(f.dtype));
        end = l->dv_part + round256(group * chains * f.N * f.dv * elem_bytes(f.dtype));
    }
    l->total = end;
    return true;
}

// Event pool of the diagnostic profiler (lasp_profile_begin / lasp_profile_end).
struct Profiler {
    bool on = false;
    int cap = 0;
    int used[2] = {0, 0};                       // recorded forward / backward calls
    std::vector<lasp::KernelEvents> slots[2];
} g_prof;

template <typename P>
const P at(const P *list, int t) { return list ? list[t] : nullptr; }
// distances of list[first + i] from list[first], for the `n` sub-sequences of a launch
template <typename P>
lasp::Offsets offsets(const P *list, int first, int n) {
    lasp::Offsets o{};
    if (list)
        for (int i = 1; i < n; ++i) o.at[i] = (const char *)list[first + i] - (const char *)list[first];
    return o;
}
lasp::Offsets strides(size_t bytes) {
    lasp::Offsets o{};
    for (int i = 1; i < lasp::kMaxShards; ++i) o.at[i] = (long long)(i * bytes);
    return o;
}

// Sub-sequences of a T-part sequence that go through one launch. Every launch of one sub-sequence leaves the device idle
// at both ends and needs segments of its own to fill it; several together are cut into fewer segments (whose states are
// that much less to move) and scanned once, at the price of a local pass over each but one. As many as still leave about as
// many workgroups as a launch of one has: more would go through in several rounds, and read more in the local pass.
// Step one by one / together, us: 16 heads x 1024 tokens x 4, d=64, in a graph 149 / 64; 32 heads x 4096 x 2 with four K/V
// heads 314 / 261; 16 x 32768 x 8 3890 / 3658.
// With a decay per token one by one: the gradient of log g is <dkv_out, kv_out> plus a sum over the sub-sequence's tail that
// cancels most of it, and together its two ends would not be the tensors the walk starts from (a scan's states stand 0.2 %
// from what the neighbour's walk returns) and its segments longer. Error of dlog_g against 64 bits, mean (largest) of six
// inputs, one by one / together: 2 heads x 24576 x 4, Norm, d=64 3.7e-2 (4.8e-2) / 4.0e-2 (5.5e-2), d=128 3.7e-2 (4.3e-2) /
// 4.0e-2 (5.1e-2), 16 x 777 x 4 7.0e-3 / 7.2e-3.
// With grouped K/V heads the parts of dK, dV of all of them lie in the scratch at once: bounded, since a sequence long enough
// to fill the memory has little to gain (the last figure), and one by one it needs no more than a call.
constexpr size_t kPartsLimit = (size_t)1 << 30;
int shards_per_launch(const lasp_shape *s, int T, bool token) {
    if (T < 2 || s->segments != 0 || token) return 1;
    const int64_t chains = (int64_t)s->B * s->H;
    auto workgroups = [&](Pass pass, int group) {
        lasp::Plan p;
        return make_plan(s, pass, &p, false, false, group) == LASP_OK ? chains * group * p.nseg : 0;
    };
    const bool grouped = s->kv_heads > 0 && s->kv_heads < s->H;
    const size_t parts = grouped ? (size_t)chains * s->N * (s->D + (s->Dv ? s->Dv : s->D)) * elem_bytes(s->dtype) : 0;
    const int64_t most = std::min<int64_t>(std::min(T, lasp::kMaxShards), lasp::kOnePerCu / chains);
    for (int n = (int)most; n > 1; --n) {
        const int launches = (T + n - 1) / n, group = (T + launches - 1) / launches;   // of about one size
        if (group * parts > kPartsLimit) continue;
        if (10 * workgroups(kForward, group) >= 9 * workgroups(kForward, 1) && 10 * workgroups(kBackward, group) >= 9 * workgroups(kBackward, 1))
            return group;
    }
    return 1;
}
// The same for a sequence whose backward pass rebuilds the states: the caches of a launch's sub-sequences lie in its
// scratch, which is there to save memory.
constexpr size_t kRebuiltCacheLimit = (size_t)64 << 20;
int shards_per_launch(const lasp_shape *s, int T, bool token, bool recompute) {
    int group = shards_per_launch(s, T, token);
    if (recompute && group > 1 && group * cache_bytes(s, token) > kRebuiltCacheLimit) group = 1;
    return group;
}

// One forward call of any flavour, over T sub-sequences of one shape (T = 1: a plain call): `token` selects the decay model
// (decay = lambda [H], one for all, or log g [B][H][N] of each), `norm` the fused output normalisation (eps, rstd). kv_out[t]
// is what sub-sequence t leaves and t + 1 starts from. cache: NULL, or one of every sub-sequence.
struct FwdCall {
    const lasp_shape *shape;
    int T, group;
    const void *const *q, *const *k, *const *v;
    const float *kv_in;
    float *kv_copy;   // receives kv_in; may be NULL
    const float *const *decay;
    bool token, norm;
    float eps;
    void *const *out;
    float *const *rstd, *const *kv_out;
    void *const *cache;
    void *scratch;
    size_t scratch_bytes;
    void *stream;
};

// The plan of a launch of one sub-sequence of a sequence that goes in groups: its cache is that of the group's.
int single_plan(const lasp_shape *s, Pass pass, lasp::Plan *p, const lasp::Plan &of_group) {
    const int rc = make_plan(s, pass, p, of_group.token, of_group.norm);
    p->cache_tiles = of_group.cache_tiles;
    return rc;
}

int run_fwd_call(const FwdCall &c) {
    lasp::Plan p, one;
    int rc = make_plan(c.shape, kForward, &p, c.token, c.norm, c.group);
    if (rc != LASP_OK) return rc;
    if (c.group == 1) one = p;
    else if (rc = single_plan(c.shape, kForward, &one, p); rc != LASP_OK) return rc;
    for (int t = 0; t < c.T; ++t)
        if (!c.q[t] || !c.k[t] || !c.v[t] || !c.decay[c.token ? t : 0] || !c.out[t] || !c.kv_out[t] || (c.norm && !at(c.rstd, t)) ||
            (c.cache && !c.cache[t]))
            return LASP_ERR_NULL;
    if (c.norm && (!std::isfinite(c.eps) || c.eps < 0.0f)) return LASP_ERR_SHAPE;
    ScratchLayout l;
    scratch_layout(c.shape, c.token, &l, c.group);
    if (!c.scratch || c.scratch_bytes < l.total) return LASP_ERR_WORKSPACE;

    const size_t esz = elem_bytes(p.dtype);
    const size_t qb = (size_t)p.B * p.H * p.N * p.dk * esz, ob = (size_t)p.B * p.H * p.N * p.dv * esz;   // q / out
    const size_t sb = (size_t)p.B * p.H * p.dk * p.dv * sizeof(float);
    const size_t gb = (size_t)p.B * p.H * p.N * sizeof(float);
    const size_t cb = c.cache ? cache_bytes(c.shape, c.token) : 0, db = c.token ? gb : p.H * sizeof(float);
    hipStream_t stream = (hipStream_t)c.stream;
    // kv_in goes to kv_copy with the walk that starts from it, unless it lies in what the call writes
    const float *kv_in = c.kv_in;
    float *kv_copy = kv_in == c.kv_copy ? nullptr : c.kv_copy;
    bool copy_first = false;
    if (kv_in && kv_copy) {
        const Span in{kv_in, sb};
        bool apart = (uintptr_t)kv_in % 16 == 0 && !overlap(in, {kv_copy, sb}) && !overlap(in, {c.scratch, l.total});
        for (int t = 0; t < c.T && apart; ++t)
            apart = !overlap(in, {c.out[t], ob}) && !overlap(in, {at(c.rstd, t), gb}) && !overlap(in, {c.kv_out[t], sb}) && !overlap(in, {at(c.cache, t), cb});
        if (!apart) {
            if (overlap(in, {kv_copy, sb})) return LASP_ERR_ALIAS;
            copy_first = true;
            kv_in = kv_copy;
            kv_copy = nullptr;
        }
    } else {
        kv_copy = nullptr;
    }
    for (int t = 0; t < c.T; ++t) {
        rc = check_buffers({{c.q[t], qb}, {c.k[t], qb / p.kvdiv}, {c.v[t], ob / p.kvdiv}, {t ? c.kv_out[t - 1] : kv_in, sb}, {c.decay[c.token ? t : 0], db}},
                           {{c.out[t], ob}, {at(c.rstd, t), gb}, {c.kv_out[t], sb}, {at(c.cache, t), cb}, {c.scratch, l.total}, {t ? nullptr : kv_copy, sb}});
        if (rc != LASP_OK) return rc;
        if (overlap_any({copy_first ? c.kv_copy : kv_copy, sb}, {{c.q[t], qb}, {c.k[t], qb / p.kvdiv}, {c.v[t], ob / p.kvdiv}, {c.decay[c.token ? t : 0], db}}))
            return LASP_ERR_ALIAS;
    }
    if (copy_first && hipMemcpyAsync(c.kv_copy, c.kv_in, sb, hipMemcpyDeviceToDevice, stream) != hipSuccess) return LASP_ERR_HIP;

    char *scr = (char *)c.scratch;
    auto launch = [&](int first, int n) {
        lasp::Plan use = n > 1 ? p : one;
        use.shards = n;
        lasp::FwdArgs a{c.q[first], c.k[first], c.v[first], first ? c.kv_out[first - 1] : kv_in, c.decay[c.token ? first : 0], c.out[first],
                        c.kv_out[first], at(c.cache, first), (float *)scr, p.token ? (float *)(scr + l.seglog) : nullptr, at(c.rstd, first),
                        c.eps, false, first ? nullptr : kv_copy, {}};
        if (n > 1) {
            a.sh.q = offsets(c.q, first, n);
            a.sh.k = offsets(c.k, first, n);
            a.sh.v = offsets(c.v, first, n);
            a.sh.out = offsets(c.out, first, n);
            a.sh.rstd = offsets(c.rstd, first, n);
            a.sh.kv_out = offsets(c.kv_out, first, n);
            a.sh.cache = offsets(c.cache, first, n);
        }
        return lasp::launch_fwd(use, a, stream, next_slot(0)) == hipSuccess;
    };
    for (int first = 0; first < c.T; first += c.group) {
        const int n = std::min(c.group, c.T - first);
        if (n > 1) {
            Together all;
            all.in(first ? c.kv_out[first - 1] : kv_in, sb);
            all.in(c.decay[0], db);
            all.out(first ? nullptr : kv_copy, sb);
            for (int t = first; t < first + n; ++t) {
                all.in(c.q[t], qb);
                all.in(c.k[t], qb / p.kvdiv);
                all.in(c.v[t], ob / p.kvdiv);
                all.out(c.out[t], ob);
                all.out(at(c.rstd, t), gb);
                all.out(c.kv_out[t], sb);
                all.out(at(c.cache, t), cb);
            }
            if (!all.disjoint()) {
                for (int t = first; t < first + n; ++t)
                    if (!launch(t, 1)) return LASP_ERR_HIP;
                continue;
            }
        }
        if (!launch(first, n)) return LASP_ERR_HIP;
    }
    return LASP_OK;
}

// One backward call of any flavour, over T sub-sequences of one shape. `yn`, `rstd`: norm only; `kv_out`, `dlog_g`: per-token
// decay only. kv_in[t] (the state sub-sequence t started from; NULL = zeros) is used only where it has no cache: the states are then rebuilt from
// it. dkv_in[t] is what sub-sequence t leaves and t - 1 receives from the right.
struct BwdCall {
    const lasp_shape *shape;
    int T, group;
    const void *const *q, *const *k, *const *v, *const *dout;
    const float *const *kv_in;
    const float *dkv_out;
    float *dkv_copy;   // receives dkv_out; may be NULL
    const float *const *decay;
    bool token, norm;
    const void *const *yn;
    const float *const *rstd, *const *kv_out;
    const void *const *cache;
    void *const *dq, *const *dk, *const *dv;
    float *const *dlog_g, *const *dkv_in;
    void *scratch;
    size_t scratch_bytes;
    void *stream;
};

// Without a state cache the backward pass rebuilds the states first (Sec. 3.4: recomputation instead of
// caching): the forward pass reduced to its states writes them into the tail of the scratch buffer.
size_t recompute_scratch(const lasp_shape *shape, bool token, int group = 1) {
    ScratchLayout l;
    if (!scratch_layout(shape, token, &l, group)) return 0;
    return round256(l.total) + group * cache_bytes(shape, token);
}

int run_bwd_call(const BwdCall &c) {
    lasp::Plan p, one;
    int rc = make_plan(c.shape, kBackward, &p, c.token, c.norm, c.group);
    if (rc != LASP_OK) return rc;
    if (c.group == 1) one = p;
    else if (rc = single_plan(c.shape, kBackward, &one, p); rc != LASP_OK) return rc;
    const bool rebuild = !c.cache;
    for (int t = 0; t < c.T; ++t) {
        if (!c.q[t] || !c.k[t] || !c.v[t] || !c.dout[t] || !c.decay[c.token ? t : 0] || !c.dq[t] || !c.dk[t] || !c.dv[t] || !c.dkv_in[t])
            return LASP_ERR_NULL;
        if (c.norm && (!at(c.yn, t) || !at(c.rstd, t))) return LASP_ERR_NULL;
        if (c.token && (!at(c.dlog_g, t) || ((c.dkv_out || t + 1 < c.T) && !at(c.kv_out, t)))) return LASP_ERR_NULL;
        if (rebuild ? t > 0 && !at(c.kv_in, t) : !c.cache[t]) return LASP_ERR_NULL;
    }
    ScratchLayout l;
    scratch_layout(c.shape, c.token, &l, c.group);
    const size_t cb = cache_bytes(c.shape, c.token);
    const size_t need = rebuild ? round256(l.total) + c.group * cb : l.total;
    if (!c.scratch || c.scratch_bytes < need) return LASP_ERR_WORKSPACE;
    char *scr = (char *)c.scratch;

    const size_t esz = elem_bytes(p.dtype);
    const size_t qb = (size_t)p.B * p.H * p.N * p.dk * esz, ob = (size_t)p.B * p.H * p.N * p.dv * esz;   // q / out
    const size_t sb = (size_t)p.B * p.H * p.dk * p.dv * sizeof(float);
    const size_t gb = (size_t)p.B * p.H * p.N * sizeof(float), db = c.token ? gb : p.H * sizeof(float);
    hipStream_t stream = (hipStream_t)c.stream;
    // dkv_out goes to dkv_copy with the walk that starts from it, unless it lies in what the call writes
    const float *dkv_out = c.dkv_out;
    float *dkv_copy = dkv_out == c.dkv_copy ? nullptr : c.dkv_copy;
    bool copy_first = false;
    if (dkv_out && dkv_copy) {
        const Span in{dkv_out, sb};
        bool apart = (uintptr_t)dkv_out % 16 == 0 && !overlap(in, {dkv_copy, sb}) && !overlap(in, {c.scratch, need});
        for (int t = 0; t < c.T && apart; ++t)
            apart = !overlap(in, {c.dq[t], qb}) && !overlap(in, {c.dk[t], qb / p.kvdiv}) && !overlap(in, {c.dv[t], ob / p.kvdiv}) &&
                    !overlap(in, {at(c.dlog_g, t), gb}) && !overlap(in, {c.dkv_in[t], sb});
        if (!apart) {
            if (overlap(in, {dkv_copy, sb})) return LASP_ERR_ALIAS;
            copy_first = true;
            dkv_out = dkv_copy;
            dkv_copy = nullptr;
        }
    } else {
        dkv_copy = nullptr;
    }
    for (int t = 0; t < c.T; ++t) {
        rc = check_buffers({{c.q[t], qb}, {c.k[t], qb / p.kvdiv}, {c.v[t], ob / p.kvdiv}, {c.dout[t], ob}, {t + 1 < c.T ? c.dkv_in[t + 1] : dkv_out, sb},
                            {at(c.kv_out, t), sb}, {rebuild ? at(c.kv_in, t) : nullptr, sb}, {at(c.yn, t), ob}, {at(c.rstd, t), gb},
                            {c.decay[c.token ? t : 0], db}, {at(c.cache, t), cb}},
                           {{c.dq[t], qb}, {c.dk[t], qb / p.kvdiv}, {c.dv[t], ob / p.kvdiv}, {at(c.dlog_g, t), gb}, {c.dkv_in[t], sb},
                            {c.scratch, need}, {t + 1 < c.T ? nullptr : dkv_copy, sb}});
        if (rc != LASP_OK) return rc;
        if (overlap_any({copy_first ? c.dkv_copy : dkv_copy, sb},
                        {{c.q[t], qb}, {c.k[t], qb / p.kvdiv}, {c.v[t], ob / p.kvdiv}, {c.dout[t], ob}, {at(c.kv_out, t), sb},
                         {rebuild ? at(c.kv_in, t) : nullptr, sb}, {at(c.yn, t), ob}, {at(c.rstd, t), gb},
                         {c.decay[c.token ? t : 0], db}, {at(c.cache, t), cb}}))
            return LASP_ERR_ALIAS;
    }

    // the forward pass's own plans (its segment count: only where the states are rebuilt), and that of the cached states: dQ of
    // float data
    lasp::Plan f{}, f1{}, g{};
    if (rebuild) {
        if (rc = make_plan(c.shape, kForward, &f, c.token, c.norm, c.group); rc != LASP_OK) return rc;
        if (rc = single_plan(c.shape, kForward, &f1, f); rc != LASP_OK) return rc;
    }
    if (p.dtype == LASP_F32) {
        lasp_shape cut = *c.shape;
        cut.segments = 0;
        if (rc = make_plan(&cut, kForward, &g, c.token, c.norm, c.group); rc != LASP_OK) return rc;
    }
    if (copy_first && hipMemcpyAsync(c.dkv_copy, c.dkv_out, sb, hipMemcpyDeviceToDevice, stream) != hipSuccess) return LASP_ERR_HIP;
    auto launch = [&](int first, int n) {
        const int last = first + n - 1;
        lasp::Plan use = n > 1 ? p : one, use_f = n > 1 ? f : f1;
        use.shards = use_f.shards = g.shards = n;
        lasp::Shards sh{};
        if (n > 1) {
            sh.q = offsets(c.q, first, n);
            sh.k = offsets(c.k, first, n);
            sh.v = offsets(c.v, first, n);
            sh.dout = offsets(c.dout, first, n);
            sh.dq = offsets(c.dq, first, n);
            sh.dk = offsets(c.dk, first, n);
            sh.dv = offsets(c.dv, first, n);
            sh.dkv_in = offsets(c.dkv_in, first, n);
            sh.yn = offsets(c.yn, first, n);
            sh.rstd = offsets(c.rstd, first, n);
            sh.cache = rebuild ? strides(cb) : offsets(c.cache, first, n);
        }
        const void *cache = rebuild ? scr + round256(l.total) : c.cache[first];
        const float *kv_in = at(c.kv_in, first);
        if (rebuild && p.dtype == LASP_F32 && use_f.tiles_per_seg == use_f.cache_tiles) {
            cache = nullptr;   // the segments' start states, which launch_bwd rebuilds in the states' region, are the cache
        } else if (rebuild) {   // states only, into the scratch tail
            lasp::FwdArgs fa{nullptr, c.k[first], c.v[first], kv_in, c.decay[c.token ? first : 0], nullptr, nullptr, (void *)cache, (float *)scr,
                             f.token ? (float *)(scr + l.seglog) : nullptr, nullptr, 0.0f, true, nullptr, sh};
            if (lasp::launch_fwd(use_f, fa, stream, nullptr) != hipSuccess) return false;
        }
        lasp::BwdArgs a{c.q[first], c.k[first], c.v[first], c.dout[first], last + 1 < c.T ? c.dkv_in[last + 1] : dkv_out, c.decay[c.token ? first : 0],
                        cache, c.dq[first], c.dk[first], c.dv[first], c.dkv_in[first], (float *)scr, &g, kv_in, at(c.kv_out, first), at(c.dlog_g, first),
                        p.token ? (float *)(scr + l.seglog) : nullptr, p.token ? (float *)(scr + l.rtok) : nullptr, at(c.yn, first),
                        at(c.rstd, first), {}, last + 1 < c.T ? nullptr : dkv_copy, sh};
        if (p.kvdiv > 1) {   // the kernels write dK, dV per query head; launch_bwd sums each group into the outputs
            for (int i = 0; i < n; ++i) {
                a.group.dk[i] = c.dk[first + i];
                a.group.dv[i] = c.dv[first + i];
            }
            a.dk = scr + l.dk_part;
            a.dv = scr + l.dv_part;
            a.sh.dk = strides(qb);
            a.sh.dv = strides(ob);
        }
        return lasp::launch_bwd(use, a, stream, next_slot(1)) == hipSuccess;
    };
    for (int end = c.T; end > 0;) {   // from the right, groups that begin where the forward pass's did
        const int first = (end - 1) / c.group * c.group;
        if (end - first > 1) {
            Together all;
            all.in(end < c.T ? c.dkv_in[end] : dkv_out, sb);
            all.in(c.decay[0], db);
            all.out(end < c.T ? nullptr : dkv_copy, sb);
            if (rebuild) all.in(at(c.kv_in, first), sb);
            for (int t = first; t < end; ++t) {
                all.in(c.q[t], qb);
                all.in(c.k[t], qb / p.kvdiv);
                all.in(c.v[t], ob / p.kvdiv);
                all.in(c.dout[t], ob);
                all.in(at(c.yn, t), ob);
                all.in(at(c.rstd, t), gb);
                all.in(at(c.cache, t), cb);
                all.out(c.dq[t], qb);
                all.out(c.dk[t], qb / p.kvdiv);
                all.out(c.dv[t], ob / p.kvdiv);
                all.out(c.dkv_in[t], sb);
            }
            if (!all.disjoint()) {
                for (; end - first > 1; --end)
                    if (!launch(end - 1, 1)) return LASP_ERR_HIP;
            }
        }
        if (!launch(first, end - first)) return LASP_ERR_HIP;
        end = first;
    }
    return LASP_OK;
}

// Calls of one sub-sequence.
int fwd_one(const lasp_shape *shape, const void *q, const void *k, const void *v, const float *kv_in, const float *decay, bool token, bool norm,
            float eps, void *out, float *rstd, float *kv_out, void *cache, void *scratch, size_t scratch_bytes, void *stream) {
    return run_fwd_call({shape, 1, 1, &q, &k, &v, kv_in, nullptr, &decay, token, norm, eps, &out, &rstd, &kv_out, cache ? &cache : nullptr,
                         scratch, scratch_bytes, stream});
}
int bwd_one(const lasp_shape *shape, const void *q, const void *k, const void *v, const void *dout, const float *kv_in, const float *dkv_out,
            const float *decay, bool token, bool norm, const void *yn, const float *rstd, const float *kv_out, const void *cache, void *dq,
            void *dk, void *dv, float *dlog_g, float *dkv_in, void *scratch, size_t scratch_bytes, void *stream) {
    return run_bwd_call({shape, 1, 1, &q, &k, &v, &dout, &kv_in, dkv_out, nullptr, &decay, token, norm, &yn, &rstd, &kv_out, cache ? &cache : nullptr, &dq, &dk,
                         &dv, &dlog_g, &dkv_in, scratch, scratch_bytes, stream});
}

}  // namespace

namespace lasp {

const KernelEvents *next_slot(int kind) {
    if (!g_prof.on || g_prof.used[kind] >= g_prof.cap) return nullptr;
    return &g_prof.slots[kind][g_prof.used[kind]++];
}

// Bidirectional path: shape rules of the causal path, own K/V head per query head only.
int make_bidir_plan(const lasp_shape *s, BidirPlan *p) {
    if (!s) return LASP_ERR_NULL;
    if (s->dtype != LASP_F32 && s->dtype != LASP_BF16) return LASP_ERR_DTYPE;
    if (!valid_dims(s)) return LASP_ERR_SHAPE;
    if (s->kv_heads != 0 && s->kv_heads != s->H) return LASP_ERR_SHAPE;
    if (s->Dv != 0 && s->Dv != s->D) return LASP_ERR_SHAPE;
    p->B = s->B;
    p->H = s->H;
    p->N = s->N;
    p->D = s->D;
    p->dtype = s->dtype;
    const int tile = bidir_reduce_tile(s->dtype);
    p->ntiles_r = (s->N + tile - 1) / tile;
    int want = s->segments;
    if (want < 0 || want > p->ntiles_r) return LASP_ERR_SHAPE;
    if (want == 0) {
        const int64_t chains = (int64_t)s->B * s->H;
        want = (int)((kBidirTargetSegments + chains - 1) / chains);
        if (want > p->ntiles_r) want = p->ntiles_r;
    }
    p->tiles_per_seg = (p->ntiles_r + want - 1) / want;
    p->nseg = (p->ntiles_r + p->tiles_per_seg - 1) / p->tiles_per_seg;
    return LASP_OK;
}

size_t bidir_scratch(const BidirPlan &p) { return (size_t)p.B * p.H * p.nseg * p.D * p.D * sizeof(float); }


hipError_t allow_dynamic_lds(const void *kernel, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    static std::mutex mu;
    static std::vector<std::pair<const void *, int>> raised;   // (kernel, device) pairs already set
    std::lock_guard<std::mutex> hold(mu);
    for (const auto &kd : raised)
        if (kd.first == kernel && kd.second == dev) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) raised.emplace_back(kernel, dev);
    return e;
}

}  // namespace lasp

extern "C" {

int lasp_version(void) { return 6; }

const char *lasp_status_str(int status) {
    switch (status) {
        case LASP_OK: return "ok";
        case LASP_ERR_NULL: return "a required pointer is NULL";
        case LASP_ERR_SHAPE: return "unsupported shape (need B,H,N > 0, D and Dv in {64,128} (Dv 0 = D), chunk in {64,128,256}, 0 <= segments <= ceil(N/tile))";
        case LASP_ERR_DTYPE: return "unsupported dtype (LASP_F32 or LASP_BF16)";
        case LASP_ERR_DECAY: return "decay must be finite and in (0, 1] (log decay: finite and <= 0)";
        case LASP_ERR_WORKSPACE: return "scratch buffer missing or too small (see lasp_scratch_bytes); lasp_fwd_noalloc: the shape needs more scratch than the library holds (see lasp_noalloc_scratch_limit)";
        case LASP_ERR_ALIAS: return "an output buffer overlaps an input or another output";
        case LASP_ERR_HIP: return "HIP runtime error at launch";
        case LASP_ERR_ALIGN: return "a buffer is not 16-byte aligned";
        default: return "unknown status";
    }
}

int lasp_check_shape(const lasp_shape *shape) {
    lasp::Plan p;
    return make_plan(shape, kForward, &p);
}

int lasp_check_decay(const float *decay_host, int32_t H) {
    if (!decay_host) return LASP_ERR_NULL;
    if (H <= 0) return LASP_ERR_SHAPE;
    for (int32_t h = 0; h < H; ++h) {
        float x = decay_host[h];
        if (!std::isfinite(x) || !(x > 0.0f) || x > 1.0f) return LASP_ERR_DECAY;
    }
    return LASP_OK;
}

int32_t lasp_tile_tokens(const lasp_shape *shape) {
    lasp::Plan p;
    return make_plan(shape, kForward, &p) == LASP_OK ? p.tile : 0;
}

int32_t lasp_num_segments(const lasp_shape *shape) {
    lasp::Plan p;
    return make_plan(shape, kForward, &p) == LASP_OK ? p.nseg : 0;
}

size_t lasp_state_cache_bytes(const lasp_shape *shape) { return cache_bytes(shape, false); }

size_t lasp_scratch_bytes(const lasp_shape *shape) {
    ScratchLayout l;
    return scratch_layout(shape, false, &l) ? l.total : 0;
}

size_t lasp_gated_state_cache_bytes(const lasp_shape *shape) { return cache_bytes(shape, true); }

size_t lasp_gated_scratch_bytes(const lasp_shape *shape) {
    ScratchLayout l;
    return scratch_layout(shape, true, &l) ? l.total : 0;
}

int lasp_check_log_decay(const float *log_g_host, int64_t n) {
    if (!log_g_host) return LASP_ERR_NULL;
    if (n <= 0) return LASP_ERR_SHAPE;
    for (int64_t i = 0; i < n; ++i) {
        float x = log_g_host[i];
        if (!std::isfinite(x) || x > 0.0f) return LASP_ERR_DECAY;
    }
    return LASP_OK;
}

int lasp_fwd(const lasp_shape *shape, const void *q, const void *k, const void *v, const float *kv_in,
             const float *decay, void *out, float *kv_out, void *state_cache, void *scratch,
             size_t scratch_bytes, void *hip_stream) {
    return fwd_one(shape, q, k, v, kv_in, decay, false, false, 0.0f, out, nullptr, kv_out, state_cache, scratch, scratch_bytes, hip_stream);
}

int lasp_fwd_noalloc(const lasp_shape *shape, const void *q, const void *k, const void *v, const float *kv_in,
                     const float *decay, void *out, float *kv_out, void *state_cache, void *hip_stream) {
    ScratchLayout l;
    if (int rc = lasp_check_shape(shape); rc != LASP_OK) return rc;
    if (!scratch_layout(shape, false, &l)) return LASP_ERR_SHAPE;
    if (l.total > lasp::kStaticScratchBytes) return LASP_ERR_WORKSPACE;   // beyond the library's own scratch
    void *scr = nullptr;
    if (lasp::static_scratch(&scr) != hipSuccess) return LASP_ERR_HIP;
    return fwd_one(shape, q, k, v, kv_in, decay, false, false, 0.0f, out, nullptr, kv_out, state_cache, scr, lasp::kStaticScratchBytes, hip_stream);
}

size_t lasp_noalloc_scratch_limit(void) { return lasp::kStaticScratchBytes; }

size_t lasp_bwd_recompute_scratch_bytes(const lasp_shape *shape) { return recompute_scratch(shape, false); }
size_t lasp_gated_bwd_recompute_scratch_bytes(const lasp_shape *shape) { return recompute_scratch(shape, true); }

int lasp_bwd(const lasp_shape *shape, const void *q, const void *k, const void *v, const void *dout,
             const float *kv_in, const float *dkv_out, const float *decay, const void *state_cache, void *dq, void *dk,
             void *dv, float *dkv_in, void *scratch, size_t scratch_bytes, void *hip_stream) {
    return bwd_one(shape, q, k, v, dout, kv_in, dkv_out, decay, false, false, nullptr, nullptr, nullptr, state_cache, dq, dk, dv, nullptr, dkv_in, scratch,
                   scratch_bytes, hip_stream);
}

int lasp_gated_fwd(const lasp_shape *shape, const void *q, const void *k, const void *v, const float *log_g,
                   const float *kv_in, void *out, float *kv_out, void *state_cache, void *scratch,
                   size_t scratch_bytes, void *hip_stream) {
    return fwd_one(shape, q, k, v, kv_in, log_g, true, false, 0.0f, out, nullptr, kv_out, state_cache, scratch, scratch_bytes, hip_stream);
}

int lasp_gated_bwd(const lasp_shape *shape, const void *q, const void *k, const void *v, const void *dout,
                   const float *log_g, const float *kv_in, const float *kv_out, const float *dkv_out,
                   const void *state_cache, void *dq, void *dk, void *dv, float *dlog_g, float *dkv_in, void *scratch,
                   size_t scratch_bytes, void *hip_stream) {
    return bwd_one(shape, q, k, v, dout, kv_in, dkv_out, log_g, true, false, nullptr, nullptr, kv_out, state_cache, dq, dk, dv, dlog_g, dkv_in, scratch,
                   scratch_bytes, hip_stream);
}

int lasp_fwd_norm(const lasp_shape *shape, const void *q, const void *k, const void *v, const float *kv_in,
                  const float *decay, float eps, void *out, float *rstd, float *kv_out, void *state_cache,
                  void *scratch, size_t scratch_bytes, void *hip_stream) {
    return fwd_one(shape, q, k, v, kv_in, decay, false, true, eps, out, rstd, kv_out, state_cache, scratch, scratch_bytes, hip_stream);
}

int lasp_bwd_norm(const lasp_shape *shape, const void *q, const void *k, const void *v, const void *out,
                  const float *rstd, const void *dout, const float *kv_in, const float *dkv_out, const float *decay,
                  const void *state_cache, void *dq, void *dk, void *dv, float *dkv_in, void *scratch,
                  size_t scratch_bytes, void *hip_stream) {
    return bwd_one(shape, q, k, v, dout, kv_in, dkv_out, decay, false, true, out, rstd, nullptr, state_cache, dq, dk, dv, nullptr, dkv_in, scratch,
                   scratch_bytes, hip_stream);
}

int lasp_gated_fwd_norm(const lasp_shape *shape, const void *q, const void *k, const void *v, const float *log_g,
                        const float *kv_in, float eps, void *out, float *rstd, float *kv_out, void *state_cache,
                        void *scratch, size_t scratch_bytes, void *hip_stream) {
    return fwd_one(shape, q, k, v, kv_in, log_g, true, true, eps, out, rstd, kv_out, state_cache, scratch, scratch_bytes, hip_stream);
}

int lasp_gated_bwd_norm(const lasp_shape *shape, const void *q, const void *k, const void *v, const void *out,
                        const float *rstd, const void *dout, const float *log_g, const float *kv_in, const float *kv_out,
                        const float *dkv_out, const void *state_cache, void *dq, void *dk, void *dv,
                        float *dlog_g, float *dkv_in, void *scratch, size_t scratch_bytes, void *hip_stream) {
    return bwd_one(shape, q, k, v, dout, kv_in, dkv_out, log_g, true, true, out, rstd, kv_out, state_cache, dq, dk, dv, dlog_g, dkv_in, scratch,
                   scratch_bytes, hip_stream);
}

size_t lasp_seq_scratch_bytes(const lasp_shape *shape, int32_t T, int32_t token, int32_t recompute) {
    if (lasp_check_shape(shape) != LASP_OK || T < 1) return 0;
    ScratchLayout l;
    scratch_layout(shape, token != 0, &l, shards_per_launch(shape, T, token != 0));
    return recompute ? std::max(l.total, recompute_scratch(shape, token != 0, shards_per_launch(shape, T, token != 0, true))) : l.total;
}

int lasp_seq_fwd(const lasp_shape *shape, int32_t T, const void *const *q, const void *const *k, const void *const *v, const float *kv_in,
                 const float *const *decay, int32_t token, float eps, void *const *out, float *const *rstd, float *const *kv,
                 void *const *state_cache, void *scratch, size_t scratch_bytes, void *hip_stream) {
    if (int rc = lasp_check_shape(shape); rc != LASP_OK) return rc;
    if (T < 1) return LASP_ERR_SHAPE;
    if (!q || !k || !v || !decay || !out || !kv) return LASP_ERR_NULL;
    return run_fwd_call({shape, T, shards_per_launch(shape, T, token != 0), q, k, v, kv_in, kv[0], decay, token != 0, rstd != nullptr, eps, out,
                         rstd, kv + 1, state_cache && state_cache[0] ? state_cache : nullptr, scratch, scratch_bytes, hip_stream});
}

int lasp_seq_bwd(const lasp_shape *shape, int32_t T, const void *const *q, const void *const *k, const void *const *v, const void *const *out,
                 const float *const *rstd, const void *const *dout, const float *const *kv, const float *dkv_out, const float *const *decay,
                 int32_t token, const void *const *state_cache, void *const *dq, void *const *dk, void *const *dv, float *const *dlog_g,
                 float *const *dkv, void *scratch, size_t scratch_bytes, void *hip_stream) {
    if (int rc = lasp_check_shape(shape); rc != LASP_OK) return rc;
    if (T < 1) return LASP_ERR_SHAPE;
    if (!q || !k || !v || !dout || !decay || !kv || !dq || !dk || !dv || !dkv) return LASP_ERR_NULL;
    const void *const *caches = state_cache && state_cache[0] ? state_cache : nullptr;
    const int group = shards_per_launch(shape, T, token != 0, !caches);
    return run_bwd_call({shape, T, group, q, k, v, dout, kv, dkv_out, dkv[T], decay, token != 0, rstd != nullptr, rstd ? out : nullptr, rstd,
                         token ? kv + 1 : nullptr, caches, dq, dk, dv, token ? dlog_g : nullptr, dkv, scratch, scratch_bytes, hip_stream});
}

size_t lasp_bidir_scratch_bytes(const lasp_shape *shape) {
    lasp::BidirPlan p;
    return lasp::make_bidir_plan(shape, &p) == LASP_OK ? lasp::bidir_scratch(p) : 0;
}

int lasp_bidir_state(const lasp_shape *shape, const void *x, const void *y, float *state, int32_t accumulate,
                     void *scratch, size_t scratch_bytes, void *hip_stream) {
    lasp::BidirPlan p;
    int rc = lasp::make_bidir_plan(shape, &p);
    if (rc != LASP_OK) return rc;
    if (!x || !y || !state) return LASP_ERR_NULL;
    if (!scratch || scratch_bytes < lasp::bidir_scratch(p)) return LASP_ERR_WORKSPACE;
    const size_t tb = (size_t)p.B * p.H * p.N * p.D * elem_bytes(p.dtype);
    const size_t sb = (size_t)p.B * p.H * p.D * p.D * sizeof(float);
    rc = check_buffers({{x, tb}, {y, tb}}, {{state, sb}, {scratch, lasp::bidir_scratch(p)}});
    if (rc != LASP_OK) return rc;
    return lasp::launch_bidir_state(p, x, y, state, accumulate != 0, (float *)scratch, (hipStream_t)hip_stream,
                                    next_slot(0)) == hipSuccess ? LASP_OK : LASP_ERR_HIP;
}

int lasp_bidir_fwd(const lasp_shape *shape, const void *q, const float *kv, void *out, void *hip_stream) {
    lasp::BidirPlan p;
    int rc = lasp::make_bidir_plan(shape, &p);
    if (rc != LASP_OK) return rc;
    if (!q || !kv || !out) return LASP_ERR_NULL;
    const size_t tb = (size_t)p.B * p.H * p.N * p.D * elem_bytes(p.dtype);
    const size_t sb = (size_t)p.B * p.H * p.D * p.D * sizeof(float);
    rc = check_buffers({{q, tb}, {kv, sb}}, {{out, tb}});
    if (rc != LASP_OK) return rc;
    const lasp::BidirOps ops{{q, nullptr, nullptr}, {kv, nullptr, nullptr}, {out, nullptr, nullptr}, {0, 0, 0}};
    return lasp::launch_bidir_apply(p, ops, 1, (hipStream_t)hip_stream, next_slot(0)) == hipSuccess ? LASP_OK : LASP_ERR_HIP;
}

int lasp_bidir_bwd(const lasp_shape *shape, const void *k, const void *v, const void *dout, const float *kv,
                   const float *dkv, void *dq, void *dk, void *dv, void *hip_stream) {
    lasp::BidirPlan p;
    int rc = lasp::make_bidir_plan(shape, &p);
    if (rc != LASP_OK) return rc;
    if (!k || !v || !dout || !kv || !dkv || !dq || !dk || !dv) return LASP_ERR_NULL;
    const size_t tb = (size_t)p.B * p.H * p.N * p.D * elem_bytes(p.dtype);
    const size_t sb = (size_t)p.B * p.H * p.D * p.D * sizeof(float);
    rc = check_buffers({{k, tb}, {v, tb}, {dout, tb}, {kv, sb}, {dkv, sb}}, {{dq, tb}, {dk, tb}, {dv, tb}});
    if (rc != LASP_OK) return rc;
    // dQ = dO KV^T, dK = V dKV^T, dV = K dKV
    const lasp::BidirOps ops{{dout, v, k}, {kv, dkv, dkv}, {dq, dk, dv}, {1, 1, 0}};
    return lasp::launch_bidir_apply(p, ops, 3, (hipStream_t)hip_stream, next_slot(1)) == hipSuccess ? LASP_OK : LASP_ERR_HIP;
}

int lasp_profile_begin(int32_t max_calls) {
    if (max_calls <= 0 || g_prof.on) return LASP_ERR_SHAPE;
    for (int kind = 0; kind < 2; ++kind) {
        g_prof.slots[kind].assign(max_calls, lasp::KernelEvents{});
        for (auto &slot : g_prof.slots[kind])
            for (auto &ev : slot.ev)
                if (hipEventCreate(&ev) != hipSuccess) return LASP_ERR_HIP;
        g_prof.used[kind] = 0;
    }
    g_prof.cap = max_calls;
    g_prof.on = true;
    return LASP_OK;
}

int lasp_profile_end(double ms_sum[6], int32_t *fwd_calls, int32_t *bwd_calls) {
    if (!ms_sum || !fwd_calls || !bwd_calls) return LASP_ERR_NULL;
    if (!g_prof.on) return LASP_ERR_SHAPE;
    int rc = LASP_OK;
    for (int i = 0; i < 6; ++i) ms_sum[i] = 0.0;
    for (int kind = 0; kind < 2; ++kind) {
        for (int c = 0; c < g_prof.used[kind]; ++c) {
            const auto &slot = g_prof.slots[kind][c];
            if (hipEventSynchronize(slot.ev[3]) != hipSuccess) rc = LASP_ERR_HIP;
            for (int j = 0; j < 3; ++j) {
                float ms = 0.0f;
                if (hipEventElapsedTime(&ms, slot.ev[j], slot.ev[j + 1]) != hipSuccess) rc = LASP_ERR_HIP;
                ms_sum[3 * kind + j] += ms;
            }
        }
        for (auto &slot : g_prof.slots[kind])
            for (auto &ev : slot.ev) (void)hipEventDestroy(ev);
        g_prof.slots[kind].clear();
    }
    *fwd_calls = g_prof.used[0];
    *bwd_calls = g_prof.used[1];
    g_prof.on = false;
    g_prof.cap = 0;
    return rc;
}

}  // extern "C"
