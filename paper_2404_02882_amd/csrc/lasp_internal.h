// Internal interface between the C-ABI host layer (lasp_api.cpp) and the HIP
// kernels (lasp_kernels.hip, lasp_walks.hip). Not installed; the public boundary is include/lasp.h.
#ifndef LASP_INTERNAL_H
#define LASP_INTERNAL_H

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

namespace lasp {

// Everything a launch needs, already validated by the host layer.
struct Plan {
    int B, H, N, D;     // D: the kernels' head dimension, max(dk, dv)
    int dk, dv;         // key (q, k) and value (v, out) dimensions as stored; the narrower one is zero-padded to D on chip
    int dtype;          // 0 = float, 1 = bfloat16
    int tile;           // tokens per kernel tile (CT)
    int ntiles;         // ceil(N / tile); only the last tile may be short
    int shards;         // sub-sequences that go through one launch, cut alike (N, ntiles, nseg, ...: of one of them)
    int nseg;           // segments per head (S)
    int tiles_per_seg;  // ceil(ntiles / nseg); the last segment may be shorter
    int scratch_segs;   // segments whose states the scratch has room for (>= nseg, unless own_states)
    int cache_tiles;    // the state cache holds the state every cache_tiles-th tile starts from, whatever `segments` a
                        // call asks for: bfloat16 2 (the backward walk takes tiles in pairs) or 1 (one by one, see
                        // cache_every_tile), float the segments of the forward pass at segments = 0 (where the walk
                        // that produces dQ starts)
    bool ragged;        // the last tile is short, or (bfloat16, backward) the last pair of tiles has only one
    bool token;         // per-token decay: `decay` of the argument structs is log g, [B][H][N]
    bool norm;          // output rows are normalised (forward epilogue, backward prologue)
    int kvdiv;          // query heads per K/V head (1 = every query head has its own)
    bool own_states;    // every workgroup of a walk computes its segment's start state itself: no local pass, no scan, no scratch
};

// Sub-sequences of one shape, each with buffers of its own, can go through the kernels in one launch (blockIdx.z), the
// segments of all of them scanned together (one lambda per head only). A kernel gets the pointers of the first and, per tensor, the distance in bytes to
// the others'. (Four at most: kernel arguments cost the host time, a launch with all distances of eight 1 us.)
constexpr int kMaxShards = 4;
struct Offsets {
    long long at[kMaxShards];
};
struct Shards {
    Offsets q, k, v, dout, cache, out, rstd, kv_out, dq, dk, dv, dkv_in, yn;
};
// What each kernel needs of it (the forward walk as kDq: dO, V, K as q, k, v, dQ as out).
struct Alone {};      // a launch of one sub-sequence: nothing
struct AloneOwn {};   // nor one whose workgroups compute their own start states
struct LocalShards {
    Offsets x, y, yn, rstd;
};
struct FwdShards {
    Offsets q, k, v, cache, out, rstd, kv_out, yn;
};
struct BwdShards {
    Offsets q, k, v, dout, cache, dq, dk, dv, dkv_in, yn, rstd;
};

#ifdef __HIPCC__
#define LASP_BOTH __host__ __device__
#else
#define LASP_BOTH
#endif
// The pieces the local pass cuts the segments of a launch into, one workgroup and one state of the scratch each: whole
// segments, or two pieces of each where whole ones would leave most of the device idle (local_pieces in lasp_rules.h). Pieces
// are numbered over all sub-sequences of the launch. (Kernels work this out: arguments cost a launch time.)
struct Pieces {
    int n;           // pieces per segment
    int tiles;       // tiles of a piece (the last of a sub-sequence may be shorter)
    int per_shard;   // pieces of a sub-sequence
    int first, end;  // the pieces that another segment's state depends on: the local pass sums these
    int base;        // the piece whose state is the scratch's first (of a chain)
    int slots;       // states of a chain in the scratch
    LASP_BOTH Pieces(bool bwd, bool two, int shards, int nseg, int tiles_per_seg, int ntiles)
        : n(two ? 2 : 1), tiles(two ? tiles_per_seg / 2 : tiles_per_seg),
          per_shard(two ? 2 * nseg - (ntiles - (nseg - 1) * tiles_per_seg > tiles ? 0 : 1) : nseg), first(bwd ? n : 0),
          end(shards * per_shard - (bwd ? 0 : per_shard - (nseg - 1) * n)), base(two ? first : 0), slots(two ? end - first : shards * nseg) {}
};

struct FwdArgs {
    const void *q, *k, *v;
    const float *kv_in;   // entering the first sub-sequence; may be null (zeros)
    const float *decay;   // lambda [H], or log g [B][H][N] with per-token decay
    void *out;
    float *kv_out;
    void *cache;          // may be null
    float *scratch;       // [B*H][shards * nseg][d_k][d_v]
    float *seglog;        // per-token decay only: [B*H][nseg], log2 of the decay over each segment
    float *rstd_out;      // norm only: [B][H][N]
    float eps;            // norm only
    bool states_only;     // rebuild the state cache only: q, out, rstd_out are not touched, kv_out may be null
    float *kv_copy;       // where kv_in is copied to, may be null
    Shards sh;
};

// Per sub-sequence, with grouped K/V heads: dk, dv [B][kv_heads][N][D].
struct GroupOut {
    void *dk[kMaxShards], *dv[kMaxShards];
};
struct BwdArgs {
    const void *q, *k, *v, *dout;
    const float *dkv_out; // entering the last sub-sequence from the right; may be null (zeros)
    const float *decay;
    const void *cache;
    void *dq, *dk, *dv;
    float *dkv_in;
    float *scratch;
    // float data only: the plan of the walk that produces dQ, one segment per cached state; and, when cache is null,
    // the state the forward pass started from
    const Plan *fwd;
    const float *kv_in;
    // per-token decay only
    const float *kv_out;  // state the forward pass returned (needed when dkv_out is given)
    float *dlog_g;        // [B][H][N]
    float *seglog;        // [B*H][nseg]
    float *rtok;          // [B*H][N] scratch: q_t.dq_t - k_t.dk_t
    // norm only: `dout` is the gradient w.r.t. the normalised output
    const void *yn;       // the normalised output the forward pass wrote
    const float *rstd;    // [B][H][N], from the forward pass
    // grouped K/V heads only (kvdiv > 1): dk, dv above are per-query-head buffers in scratch,
    // summed over each group into these
    GroupOut group;
    float *dkv_copy;      // where dkv_out is copied to, may be null
    Shards sh;
};

// Optional event recorder: when non-null, launch_* records ev[0] before the
// local pass, ev[1] after it, ev[2] after the scan and ev[3] after the walk.
struct KernelEvents {
    hipEvent_t ev[4];
};

// Raises the dynamic LDS limit of `kernel` (its host-side address) to `bytes` when that exceeds the 64 KB
// default. The attribute belongs to the kernel and the device's loaded module, so the runtime is asked
// once per (kernel, device) pair; later calls are a table lookup. Thread-safe.
hipError_t allow_dynamic_lds(const void *kernel, size_t bytes);

// The library's own scratch for lasp_fwd_noalloc: a file-scope device array of kStaticScratchBytes
// (32 MiB: 512 float [128][128] segment states; an automatic bfloat16 plan of up to 256 heads takes half of it). static_scratch() returns
// its address on the current device (resolved once per device).
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
hipError_t static_scratch(void **ptr);

// Tile length used for a (dtype, chunk, D) combination.
int tile_tokens(int dtype, int chunk, int D);

// Over the segments of every head, in place in `states` ([chain][nseg][d_k][d_v]): local states -> start states.
hipError_t launch_scan(const Plan &p, bool bwd, float *states, const float *boundary, const float *decay, const float *seglog,
                       hipStream_t s);
hipError_t launch_dlg(const Plan &p, const BwdArgs &a, hipStream_t s);
// dk, dv [K/V head] = sum of the parts of its query heads
hipError_t launch_group_sum(const Plan &p, const BwdArgs &a, hipStream_t s);

// The passes for one data type and one (d_k, d_v), each in a translation unit of its own (lasp_walks.hip).
#define LASP_PASSES(NAME)                                                                         \
    hipError_t fwd_##NAME(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke); \
    hipError_t bwd_##NAME(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke);
LASP_PASSES(f32_64) LASP_PASSES(f32_128) LASP_PASSES(f32_64_128) LASP_PASSES(f32_128_64)
LASP_PASSES(bf16_64) LASP_PASSES(bf16_128) LASP_PASSES(bf16_64_128) LASP_PASSES(bf16_128_64)
#undef LASP_PASSES

hipError_t launch_fwd(const Plan &p, const FwdArgs &a, hipStream_t stream, const KernelEvents *ke);
hipError_t launch_bwd(const Plan &p, const BwdArgs &a, hipStream_t stream, const KernelEvents *ke);


// Bidirectional (unmasked) path: O = Q (K^T V).
struct BidirPlan {
    int B, H, N, D, dtype;
    int ntiles_r;        // ceil(N / reduce tile)
    int nseg;            // segments per head of the state reduction (partial sums in scratch)
    int tiles_per_seg;   // ceil(ntiles_r / nseg); every segment non-empty
};
// Up to three products Out = X S (trans == 0) or X S^T (trans != 0), S [B*H][D][D] float.
struct BidirOps {
    const void *x[3];
    const float *s[3];
    void *out[3];
    int trans[3];
};
// The same over n <= kMaxShards sub-sequences of any lengths (host arrays of n). A sum of the states of all of them:
struct BidirSums {
    int n;
    const int *ntok;
    const void *const *x, *const *y;
    float *state;
    int accumulate;
    float *part;
    void *const *dq;    // with y = dO: also dQ = dO kv^T; or null
    const float *kv;
};
// and products of each with the same state.
struct BidirProducts {
    int n;
    const int *ntok;
    int nops;
    const void *const *x[3];
    const float *s[3];
    void *const *out[3];
    int trans[3];
};
constexpr int kBidirTargetWorkgroups = 512;   // products: two 4-wave workgroups per CU
constexpr int kBidirTargetSegments = 256;     // reduction: one partial sum per CU (fewer partials to write and add)
int bidir_reduce_tile(int dtype);
int bidir_product_tile(int dtype);
// events: ev[0]..ev[1] the reduction, ev[1]..ev[2] the sum of the partials
hipError_t launch_bidir_state(const BidirPlan &p, const void *x, const void *y, float *state, int accumulate, float *part,
                              hipStream_t stream, const KernelEvents *ke);
hipError_t launch_bidir_sums(const BidirPlan &p, const BidirSums &a, hipStream_t stream, const KernelEvents *ke);
// events: ev[2]..ev[3] the product kernel
hipError_t launch_bidir_products(const BidirPlan &p, const BidirProducts &a, hipStream_t stream, const KernelEvents *ke);
hipError_t launch_bidir_apply(const BidirPlan &p, const BidirOps &ops, int nops, hipStream_t stream, const KernelEvents *ke);

}  // namespace lasp
#endif
