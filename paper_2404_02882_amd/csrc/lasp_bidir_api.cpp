// C-ABI host layer of whole bidirectional sequences (lasp_bidir_seq_*): the loops over the sub-sequences, several of them a
// launch where their buffers allow it. No device memory is allocated or freed here and nothing synchronises.
#include "../../include/lasp.h"

#include <algorithm>

#include "lasp_checks.h"
#include "lasp_internal.h"
#include "lasp_rules.h"

namespace {

using lasp::BidirPlan;
using lasp::kMaxShards;
using lasp::Span;

// One plan for `n` sub-sequences: the reduction's segments are cut over the tiles of all of them.
BidirPlan group_plan(const lasp_shape *shapes, int n) {
    BidirPlan p;
    lasp::make_bidir_plan(shapes, &p);
    if (n == 1) return p;
    const int tile = lasp::bidir_reduce_tile(p.dtype);
    p.ntiles_r = 0;
    for (int t = 0; t < n; ++t) p.ntiles_r += (shapes[t].N + tile - 1) / tile;
    const int64_t chains = (int64_t)p.B * p.H;
    const int want = (int)std::min<int64_t>((lasp::kBidirTargetSegments + chains - 1) / chains, p.ntiles_r);
    p.tiles_per_seg = (p.ntiles_r + want - 1) / want;
    p.nseg = (p.ntiles_r + p.tiles_per_seg - 1) / p.tiles_per_seg;
    return p;
}

// Sub-sequences of a launch: as many as there is room for, but one by one where the caller chose the segments of each.
int group_size(const lasp_shape *shapes, int T) { return shapes[0].segments != 0 ? 1 : std::min(T, kMaxShards); }

// Whether dQ comes with the sum over the first `n` sub-sequences (all but the last launches take as many).
bool dq_with_sum(const lasp_shape *shapes, int n) {
    const BidirPlan p = group_plan(shapes, n);
    const int tile = lasp::bidir_product_tile(p.dtype);
    int tiles = 0;
    for (int t = 0; t < n; ++t) tiles += (shapes[t].N + tile - 1) / tile;
    const long long chains = (long long)p.B * p.H, three = lasp::blocks_time(tiles, 3 * chains, lasp::kBidirTargetWorkgroups),
                    two = lasp::blocks_time(tiles, 2 * chains, lasp::kBidirTargetWorkgroups);
    return lasp::dq_with_sum(p.dtype == LASP_BF16, p.D, chains, p.tiles_per_seg, p.nseg, three - two);
}

int check_shapes(const lasp_shape *shapes, int32_t T) {
    if (!shapes) return LASP_ERR_NULL;
    if (T < 1) return LASP_ERR_SHAPE;
    for (int t = 0; t < T; ++t) {
        BidirPlan p;
        if (int rc = lasp::make_bidir_plan(shapes + t, &p); rc != LASP_OK) return rc;
        if (shapes[t].B != shapes[0].B || shapes[t].H != shapes[0].H || shapes[t].D != shapes[0].D || shapes[t].dtype != shapes[0].dtype ||
            shapes[t].segments != shapes[0].segments)
            return LASP_ERR_SHAPE;
    }
    return LASP_OK;
}

size_t scratch_for(const lasp_shape *shapes, int T) {
    size_t need = 0;
    const int group = group_size(shapes, T);
    for (int t = 0; t < T; ++t) need = std::max(need, lasp::bidir_scratch(group_plan(shapes + t, 1)));   // one by one
    for (int t = 0; t < T; t += group) need = std::max(need, lasp::bidir_scratch(group_plan(shapes + t, std::min(group, T - t))));
    return need;
}

struct Sizes {
    size_t token, state;   // bytes of a token tensor of sub-sequence t (per token), of a state
    explicit Sizes(const lasp_shape &s)
        : token((size_t)s.B * s.H * s.D * lasp::elem_bytes(s.dtype)), state((size_t)s.B * s.H * s.D * s.D * sizeof(float)) {}
};

// Reduction over all sub-sequences, `group` of them a launch; dq: also the products with kv (see BidirSums).
bool sums(const lasp_shape *shapes, int T, int group, const void *const *x, const void *const *y, float *state, void *scratch,
          void *const *dq, const float *kv, hipStream_t s, int kind) {
    for (int t = 0; t < T; t += group) {
        const int n = std::min(group, T - t);
        int ntok[kMaxShards];
        for (int i = 0; i < n; ++i) ntok[i] = shapes[t + i].N;
        const lasp::BidirSums a{n, ntok, x + t, y + t, state, t > 0, (float *)scratch, dq ? dq + t : nullptr, kv};
        if (lasp::launch_bidir_sums(group_plan(shapes + t, n), a, s, lasp::next_slot(kind)) != hipSuccess) return false;
    }
    return true;
}
struct Product {
    const void *const *x;
    const float *state;
    void *const *out;
    int trans;
};
bool products(const lasp_shape *shapes, int T, int group, std::initializer_list<Product> ops, hipStream_t s, int kind) {
    for (int t = 0; t < T; t += group) {
        const int n = std::min(group, T - t);
        int ntok[kMaxShards];
        for (int i = 0; i < n; ++i) ntok[i] = shapes[t + i].N;
        lasp::BidirProducts a{n, ntok, 0, {}, {}, {}, {}};
        for (const Product &op : ops) {
            a.x[a.nops] = op.x + t;
            a.s[a.nops] = op.state;
            a.out[a.nops] = op.out + t;
            a.trans[a.nops++] = op.trans;
        }
        if (lasp::launch_bidir_products(group_plan(shapes + t, n), a, s, lasp::next_slot(kind)) != hipSuccess) return false;
    }
    return true;
}

}  // namespace

extern "C" {

size_t lasp_bidir_seq_scratch_bytes(const lasp_shape *shapes, int32_t T) {
    return check_shapes(shapes, T) == LASP_OK ? scratch_for(shapes, T) : 0;
}

int lasp_bidir_seq_fwd(const lasp_shape *shapes, int32_t T, const void *const *q, const void *const *k, const void *const *v,
                       float *kv, void *const *out, void *scratch, size_t scratch_bytes, void *hip_stream) {
    if (int rc = check_shapes(shapes, T); rc != LASP_OK) return rc;
    if (!q || !k || !v || !out) return LASP_ERR_NULL;
    for (int t = 0; t < T; ++t)
        if (!q[t] || !k[t] || !v[t] || !out[t] || !kv) return LASP_ERR_NULL;
    const size_t need = scratch_for(shapes, T);
    if (!scratch || scratch_bytes < need) return LASP_ERR_WORKSPACE;
    const Sizes b(shapes[0]);
    lasp::Together all;
    all.in(kv, b.state);
    for (int t = 0; t < T; ++t) {
        const size_t tb = b.token * shapes[t].N;
        // (the sum and the partial sums are written before the products read their inputs)
        if (int rc = lasp::check_buffers({{q[t], tb}, {k[t], tb}, {v[t], tb}}, {{kv, b.state}, {scratch, need}}); rc != LASP_OK) return rc;
        if (int rc = lasp::check_buffers({{q[t], tb}, {kv, b.state}}, {{out[t], tb}}); rc != LASP_OK) return rc;
        all.in(q[t], tb);
        all.out(out[t], tb);
    }
    const int group = group_size(shapes, T);
    hipStream_t s = (hipStream_t)hip_stream;
    if (!sums(shapes, T, group, k, v, kv, scratch, nullptr, nullptr, s, 0)) return LASP_ERR_HIP;
    // (outputs that lie in another sub-sequence's queries: one after the other)
    return products(shapes, T, all.disjoint() ? group : 1, {{q, kv, out, 0}}, s, 0) ? LASP_OK : LASP_ERR_HIP;
}

int lasp_bidir_seq_bwd(const lasp_shape *shapes, int32_t T, const void *const *q, const void *const *k, const void *const *v,
                       const void *const *dout, const float *kv, float *dkv, void *const *dq, void *const *dk, void *const *dv,
                       void *scratch, size_t scratch_bytes, void *hip_stream) {
    if (int rc = check_shapes(shapes, T); rc != LASP_OK) return rc;
    if (!q || !k || !v || !dout || !dq || !dk || !dv) return LASP_ERR_NULL;
    for (int t = 0; t < T; ++t)
        if (!q[t] || !k[t] || !v[t] || !dout[t] || !kv || !dkv || !dq[t] || !dk[t] || !dv[t]) return LASP_ERR_NULL;
    const size_t need = scratch_for(shapes, T);
    if (!scratch || scratch_bytes < need) return LASP_ERR_WORKSPACE;
    const Sizes b(shapes[0]);
    lasp::Together all;
    all.in(kv, b.state);
    all.out(dkv, b.state);
    all.out(scratch, need);
    for (int t = 0; t < T; ++t) {
        const size_t tb = b.token * shapes[t].N;
        if (int rc = lasp::check_buffers({{q[t], tb}, {k[t], tb}, {v[t], tb}, {dout[t], tb}, {kv, b.state}}, {{dkv, b.state}, {scratch, need}});
            rc != LASP_OK)
            return rc;
        if (int rc = lasp::check_buffers({{k[t], tb}, {v[t], tb}, {dout[t], tb}, {kv, b.state}, {dkv, b.state}}, {{dq[t], tb}, {dk[t], tb}, {dv[t], tb}});
            rc != LASP_OK)
            return rc;
        for (const void *x : {q[t], k[t], v[t], dout[t]}) all.in(x, tb);
        for (const void *x : {dq[t], dk[t], dv[t]}) all.out(x, tb);
    }
    const int group = group_size(shapes, T);
    hipStream_t s = (hipStream_t)hip_stream;
    const Product of_q{dout, kv, dq, 1}, of_k{v, dkv, dk, 1}, of_v{k, dkv, dv, 0};   // dQ = dO KV^T, dK = V dKV^T, dV = K dKV
    // Where a gradient takes the place of something that is still read then (dQ that of Q, say): all three behind the sum, one
    // sub-sequence after the other.
    const bool apart = all.disjoint();
    const bool ok = apart && dq_with_sum(shapes, std::min(group, T))
                        ? sums(shapes, T, group, q, dout, dkv, scratch, dq, kv, s, 1) && products(shapes, T, group, {of_k, of_v}, s, 1)
                        : sums(shapes, T, group, q, dout, dkv, scratch, nullptr, nullptr, s, 1) &&
                              products(shapes, T, apart ? group : 1, {of_q, of_k, of_v}, s, 1);
    return ok ? LASP_OK : LASP_ERR_HIP;
}

}  // extern "C"
