// HIP kernels (gfx950 / CDNA4) for chunked causal linear attention with decay:
// the per-device hot path of LASP (arxiv 2404.02882, Alg. 2 forward, Alg. 3
// backward).
//
// Parallel structure. One head's sub-sequence is a serial recurrence over
// tiles, and there can be as few as 16 heads, so every head is cut into
// `nseg` segments of consecutive tiles that run as independent workgroups:
//   1. k_local : each segment accumulates its local state from zero
//                (forward: sum lambda^(len-s) k_s v_s^T; backward: sum
//                lambda^s q_s do_s^T), reading only K,V (or Q,dO).
//   2. k_scan  : an elementwise scan over the segments of a head turns the
//                local states into the state each segment starts from
//                (KV_t = lambda^len KV_{t-1} + local, the state update of
//                Sec. 3.2 taken over a whole segment).
//   3. k_fwd / k_bwd8p, k_bwdkv : each segment walks its tiles with the
//                d x d state held in registers: intra-chunk left product,
//                inter-chunk right product, state update (Alg. 2 / Alg. 3 per
//                tile). Backward: k_bwd8p for bfloat16 (one cached state per
//                pair of tiles); float: dQ by k_fwd over dO, V, K, then k_bwdkv
//                for dK and dV.
// Short sequences need only step 3: with few tiles in front of it a workgroup
// takes the state through them itself (Start kOwn, own_states in lasp_rules.h).
// Every kernel is instantiated for a decay model (lasp_device.h): one lambda
// per head, or a decay per token (general recurrent form of App. A.4), which
// adds k_dlg for the gradient of the log decay; optionally with the output
// normalisation fused (forward epilogue, backward prologue); and, where the key
// and value dimensions differ, for the row widths of the key-side and value-side
// tensors (the narrower rows are zero-padded on their way to LDS).
// This is the paper's "intra parts in parallel, inter parts in sequence"
// (Alg. 2) folded onto one GPU; there are no atomics, so results are
// bit-reproducible.
//
// Wave tiling. A workgroup has D/32 waves, or two groups of as many (k_fwd8 and
// the backward walks); wave w of a group owns the 32-wide column block
// w of every [.][D] output tile and of the state, so the state tile it holds in
// MFMA accumulator layout can be fed back as the B operand of the next product
// without leaving registers (the contraction index is permuted identically on
// the A side). All products use 32x32 MFMA tiles: v_mfma_f32_32x32x16_bf16 for
// both data types, float data as three bfloat16 parts (WalkElem, lasp_device.h);
// accumulation and the state are always fp32.
#include <hip/hip_runtime.h>

#include "lasp_internal.h"
#include "lasp_rules.h"
#include "lasp_device.h"

namespace lasp {

// Grouped K/V heads: query heads h*kvdiv .. h*kvdiv+kvdiv-1 of a batch entry share K/V head h. The
// kernels index every token tensor by the query-head chain (b*H + h); K and V pointers are moved once,
// at kernel entry, by the distance between the chain's own slot and its K/V head's slot.
DEVI ptrdiff_t kv_shift(int chain, int H, int kvdiv, int ntok, int width) {
    const int kvchain = (chain / H) * (H / kvdiv) + (chain % H) / kvdiv;
    return (ptrdiff_t)(kvchain - chain) * ntok * width;
}
// Where a walk takes its segment's start state from: a state that the forward pass kept (float dQ), its slot as k_scan left
// it, the boundary state carried over the local states of the segments before (start_state), or the boundary state taken
// through the tiles of those segments by the workgroup itself, which needs no local pass and no scratch.
enum Start { kKept = -1, kScanned = 0, kCarried = 1, kOwn = 2, kCarriedPieces = 3 };   // (the last: over two pieces a segment)
// First element of tile `t` (CT tokens) of a chain in a token tensor whose rows hold `width` elements.
DEVI size_t tile_off(int chain, int ntok, int t, int CT, int width) {
    return ((size_t)chain * ntok + (size_t)t * CT) * width;
}

// ---------------------------------------------------------------------------
// k_local: local state of a segment, or of a piece of one (Pieces), from zero.
//   forward : local = sum_s lambda^(len - s) k_s v_s^T            (X = K, Y = V)
//   backward: local = sum_s lambda^s q_s do_s^T                    (X = Q, Y = dO)
// This is the state update of Alg. 2 / the dKV update of Alg. 3 unrolled over the segment's tiles: every
// token's weight is taken relative to the segment's edge (forward: its end, backward: its start) as
// (decay between the edge and the token's tile) x (the token's weight inside its tile), so the
// accumulators are plain sums and are never rescaled.
// The row weight is applied to the Y fragments (shared by all row blocks).
// ---------------------------------------------------------------------------
// NORM (backward only): Y is dY, the gradient w.r.t. the normalised output; the tile is turned into dO
// on its way to LDS from the normalised output `yn` and `rstd` ([chain][token]).
// RAGGED: the sub-sequence's last tile may be short (or missing from the last pair of tiles, k_bwd8p); without
// it every row count is CT and known at compile time.
// WX, WY: elements per row of X and Y in memory (<= D; narrower rows are zero-padded on their way to LDS,
// which serves key and value dimensions that differ).
// G: groups of D/32 waves, each with its share of the state's rows (see run_local).
template <typename T, int CT, int D, bool BWD, bool TOKEN, bool RAGGED, bool NORM, int WX, int WY, typename SH, int G>
__global__ __launch_bounds__(D * 2 * G, 2) void k_local(const T *__restrict__ X, const T *__restrict__ Y,
                                                  const float *__restrict__ decay, float *__restrict__ scratch,
                                                  float *__restrict__ seglog, int H, int ntiles, int segs,
                                                  int tiles_per_seg, int ntok, int kvdiv, const T *__restrict__ yn,
                                                  const float *__restrict__ rstd, SH sh) {
    static_assert(!NORM || BWD, "the Norm prologue belongs to the backward pass");
    using E = WalkElem<T>;
    constexpr int NT = D * 2 * G, LDD = walk_ld<T, D>(), DB = D / 32 / G, NKS = CT / E::KSTEP, TILE = walk_tile<T>(CT, LDD);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t *sX = (bf16_t *)smem;
    bf16_t *sY = sX + TILE;
    float *pw = (float *)(sY + TILE);

    constexpr bool SHARED = is_shared<SH>;
    const int chain = blockIdx.y, shard = SHARED ? blockIdx.z : 0;
    const Pieces pc(BWD, segs < 0, SHARED ? gridDim.z : 1, segs < 0 ? -segs : segs, tiles_per_seg, ntiles);   // (segs < 0: two pieces a segment)
    const int seg = blockIdx.x + (SHARED ? 0 : pc.first), piece = shard * pc.per_shard + seg;
    if (SHARED && (piece < pc.first || piece >= pc.end)) return;   // (of several sub-sequences: the grid has them all)
    const size_t slot = (size_t)chain * pc.slots + (piece - pc.base);
    const int t0 = seg * pc.tiles;
    const int t1 = min(t0 + pc.tiles, ntiles);
    const int w8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = w8 % (D / 32);  // wave index, scalar; its column block
    const int a0 = 32 * DB * (w8 / (D / 32));   // first of its state rows
    Lane ln = fresh_lane();
    if constexpr (SHARED) {
        if (shard) {
            X = at_shard(X, sh.x, shard);
            Y = at_shard(Y, sh.y, shard);
            if constexpr (NORM) {
                yn = at_shard(yn, sh.yn, shard);
                rstd = at_shard(rstd, sh.rstd, shard);
            }
        }
    }
    if (!BWD) {  // forward: X, Y are K, V
        X += kv_shift(chain, H, kvdiv, ntok, WX);
        Y += kv_shift(chain, H, kvdiv, ntok, WY);
    }
    auto xoff = [&](int t) { return tile_off(chain, ntok, t, CT, WX); };
    auto yoff = [&](int t) { return tile_off(chain, ntok, t, CT, WY); };
    const int ntl = t1 - t0;
    auto tile_of = [&](int n) { return BWD ? t1 - 1 - n : t0 + n; };
    // the first tile is requested before anything else so that its latency covers the set-up
    // rows of tile `t` that exist: the last tile of a sub-sequence may be short
    auto nvalid = [&](int t) { return RAGGED ? min(CT, ntok - t * CT) : CT; };
    // One lambda per head, forward: the weights run from the segment's end, so where a sub-sequence ends inside a tile its
    // last segment is cut into tiles from the end, and the first of them is the one that lacks rows (END_CUT).
    constexpr bool END_CUT = RAGGED && !BWD;
    static_assert(!END_CUT || (SHARED && !TOKEN), "alone, the forward pass does not sum over its last segment");
    const int gap = END_CUT ? t1 * CT - min(t1 * CT, ntok) : 0;   // rows the first tile lacks
    TileMover<T, CT, D, NT, true> mx, my;   // streaming (non-temporal) loads
    NormTile<T, CT, D, NT, WY> mn;   // the normalised output has the rows of Y (= dY)
    const float *rstd_c = rstd + (size_t)chain * ntok;
    if constexpr (!TOKEN) {   // (the per-token-decay path walks the tiles in the other order)
        if constexpr (END_CUT) {
            X -= gap * WX;
            Y -= gap * WY;
            mx.template load_tail_w<WX>(X + xoff(t0), gap);
            my.template load_tail_w<WY>(Y + yoff(t0), gap);
        } else {
            mx.template load_w<WX>(X + xoff(tile_of(0)), nvalid(tile_of(0)));
            my.template load_w<WY>(Y + yoff(tile_of(0)), nvalid(tile_of(0)));
        }
        if constexpr (NORM) mn.load(yn + yoff(tile_of(0)), rstd_c + (size_t)tile_of(0) * CT, nvalid(tile_of(0)));
    }
    f32x16 st[DB];
#pragma unroll
    for (int ab = 0; ab < DB; ++ab) st[ab] = f32x16{0};
    // Float data: the five small terms of every product are summed apart for the length of the segment.
    f32x16 low[DB];
    auto add_tile = [&](const typename E::frag(&y)[NKS]) __attribute__((always_inline)) {
        if constexpr (E::PLANES == 3)
            pipelined_flat<DB * NKS, 1>([&](int i) { return E::ld_ks(ln, sX, LDD, (i % NKS) * E::KSTEP, a0 + 32 * (i / NKS)); },
                                        [&](int i, const typename E::frag &x) {
                                            st[i / NKS] = E::mfma_high(x, y[i % NKS], st[i / NKS]);
                                            low[i / NKS] = E::mfma_low(x, y[i % NKS], low[i / NKS]);
                                        });
    };
    if constexpr (E::PLANES == 3) {
#pragma unroll
        for (int ab = 0; ab < DB; ++ab) low[ab] = f32x16{0};
    }

    if constexpr (TOKEN) {
        // `decay` is log g, [chain][token]. The sum over the segment's tokens is taken walking AWAY from the
        // edge the weights refer to (forward: tiles descending from the segment's end, weight = decay over
        // the tokens after it; backward: tiles ascending from its start, weight = decay up to and including
        // it), so a token's weight is 2^(decay of the tiles already done + its weight inside its tile) and
        // the accumulators are never rescaled (same sum as the tile recursion of Alg. 2 / Alg. 3 unrolled).
        const TokenDecay<T, CT> dec(pw);
        const float *lg = decay + (size_t)chain * ntok;
        auto tile_at = [&](int n) { return BWD ? t0 + n : t1 - 1 - n; };
        mx.template load_w<WX>(X + xoff(tile_at(0)), nvalid(tile_at(0)));
        my.template load_w<WY>(Y + yoff(tile_at(0)), nvalid(tile_at(0)));
        if constexpr (NORM) mn.load(yn + yoff(tile_at(0)), rstd_c + (size_t)tile_at(0) * CT, nvalid(tile_at(0)));
        typename TokenDecay<T, CT>::LogG lgreg = TokenDecay<T, CT>::fetch(lg + (size_t)tile_at(0) * CT, nvalid(tile_at(0)));
        float base = 0.0f;   // log2 decay of the tiles already done (kept by the wave that fills the tables)
        for (int n = 0; n < ntl; ++n) {
            __syncthreads();
            ln = fresh_lane();
            if constexpr (NORM) mn.apply(my);
            mx.store(sX, LDD);
            my.store(sY, LDD);
            base += dec.fill(lgreg, base);
            __syncthreads();
            if (n + 1 < ntl) {
                const int tn = tile_at(n + 1);
                mx.template load_w<WX>(X + xoff(tn), nvalid(tn));
                my.template load_w<WY>(Y + yoff(tn), nvalid(tn));
                if constexpr (NORM) mn.load(yn + yoff(tn), rstd_c + (size_t)tn * CT, nvalid(tn));
                lgreg = TokenDecay<T, CT>::fetch(lg + (size_t)tn * CT, nvalid(tn));
            }
            auto weigh = [&](const typename E::frag &f, int ks) { return BWD ? dec.weigh_upto(ln, f, ks) : dec.template weigh_after<true>(ln, f, ks); };
            if constexpr (E::PLANES == 3) {
                typename E::frag yd[NKS];
                unsigned lows = 0;
                auto weigh_all = [&](auto edge) __attribute__((always_inline)) {
                    constexpr bool EDGE = decltype(edge)::value;
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks) {
                        const typename E::frag y = E::ld_ks(ln, sY, LDD, ks * E::KSTEP, 32 * w);
                        if constexpr (BWD) yd[ks] = dec.template weigh_upto<EDGE>(ln, y, ks, &lows);
                        else yd[ks] = dec.template weigh_after<true, EDGE>(ln, y, ks, &lows);
                    }
                };
                weigh_all(std::false_type{});
                if (__builtin_expect(E::edge(lows), 0)) weigh_all(std::true_type{});
                add_tile(yd);
                continue;
            }
            struct Step {
                typename E::frag y;
                typename E::frag x[DB];
            };
            if constexpr (E::PLANES == 1) pipelined<NKS>(
                [&](int ks) {
                    Step f;
                    f.y = E::ld_ks(ln, sY, LDD, ks * E::KSTEP, 32 * w);
#pragma unroll
                    for (int ab = 0; ab < DB; ++ab) f.x[ab] = E::ld_ks(ln, sX, LDD, ks * E::KSTEP, a0 + 32 * ab);
                    return f;
                },
                [&](int ks, const Step &f) {
                    const typename E::frag yd = weigh(f.y, ks);
#pragma unroll
                    for (int ab = 0; ab < DB; ++ab) st[ab] = E::mfma(f.x[ab], yd, st[ab]);
                });
        }
        // log2 of the product of g over the segment, for the scan
        if (threadIdx.x == 0) seglog[slot] = base;
    } else {
    const float lam = decay[chain % H];
    fill_pow_table<CT>(pw, lam);
    const GeoWeights<T> geo(lam);
    const double lamC = pow_n(lam, CT);
    for (int n = 0; n < ntl; ++n) {
        __syncthreads();  // previous tile fully consumed (and pw visible on the first pass)
        ln = fresh_lane();
        if constexpr (NORM) mn.apply(my);
        mx.store(sX, LDD);
        // Token weight relative to the whole segment, so the accumulators are never rescaled:
        // forward lambda^(tokens after it in the segment), backward lambda^(its 1-based position).
        const float tile_factor = (float)pow_n(lamC, ntl - 1 - n);  // tiles between this one and the segment edge
        if constexpr (E::PLANES == 3) my.store_weighted(sY, LDD, [&](int row) { return tile_factor * pw[BWD ? row + 1 : CT - 1 - row]; });
        else my.store(sY, LDD);
        __syncthreads();
        if (n + 1 < ntl) {
            // (never the tile that lacks rows, which was requested first)
            mx.template load_w<WX>(X + xoff(tile_of(n + 1)), CT);
            my.template load_w<WY>(Y + yoff(tile_of(n + 1)), CT);
            if constexpr (NORM) mn.load(yn + yoff(tile_of(n + 1)), rstd_c + (size_t)tile_of(n + 1) * CT);
        }
        // bfloat16: the weight factors as (tile factor) * (table entry of the lane's first element) * g[e].
        auto weight_of = [&](int ks) {
            const int k_first = ks * E::KSTEP + E::KH * ln.h;  // lane's first token of this fragment
            return tile_factor * (BWD ? pw[k_first + 1] : pw[CT - E::KH - k_first]);
        };
        if constexpr (E::PLANES == 3) {
            typename E::frag y[NKS];   // already weighted
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) y[ks] = E::ld_ks(ln, sY, LDD, ks * E::KSTEP, 32 * w);
            add_tile(y);
        } else if constexpr (NKS * (1 + DB) * sizeof(typename E::frag) <= 80 * 4) {
            // small tiles: request every operand fragment at once (one exposed LDS latency per tile)
            typename E::frag yf[NKS], xf[NKS][DB];
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                yf[ks] = E::ld_ks(ln, sY, LDD, ks * E::KSTEP, 32 * w);
#pragma unroll
                for (int ab = 0; ab < DB; ++ab) xf[ks][ab] = E::ld_ks(ln, sX, LDD, ks * E::KSTEP, a0 + 32 * ab);
            }
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const typename E::frag yd = E::scale_geo(yf[ks], weight_of(ks), BWD ? geo.upto : geo.after);
#pragma unroll
                for (int ab = 0; ab < DB; ++ab) st[ab] = E::mfma(xf[ks][ab], yd, st[ab]);
            }
        } else {
            struct Step {
                typename E::frag y;
                typename E::frag x[DB];
            };
            pipelined<NKS>(
                [&](int ks) {
                    Step f;
                    f.y = E::ld_ks(ln, sY, LDD, ks * E::KSTEP, 32 * w);
#pragma unroll
                    for (int ab = 0; ab < DB; ++ab) f.x[ab] = E::ld_ks(ln, sX, LDD, ks * E::KSTEP, a0 + 32 * ab);
                    return f;
                },
                [&](int ks, const Step &f) {
                    const typename E::frag yd = E::scale_geo(f.y, weight_of(ks), BWD ? geo.upto : geo.after);
#pragma unroll
                    for (int ab = 0; ab < DB; ++ab) st[ab] = E::mfma(f.x[ab], yd, st[ab]);
                });
        }
    }
    }
    if constexpr (E::PLANES == 3) {
#pragma unroll
        for (int ab = 0; ab < DB; ++ab) st[ab] += low[ab];
    }
    if constexpr (G == 1) state_store_w<D, WX, WY>(ln, st, scratch + slot * WX * WY, w);
    else state_store_w<D, D, D, DB>(ln, st, scratch + slot * D * D + a0 * D, w);
}

// ---------------------------------------------------------------------------
// k_fwd: one segment of one head, tiles ascending (Alg. 2 per tile):
//   P      = (Q K^T) (.) M                       masked scores, via LDS
//   O      = P V + Lambda (Q KV_{t-1})           intra + inter
//   KV_t   = lambda^CT KV_{t-1} + (lambda^CT Lambda^-1 K)^T V
// The state KV_{t-1} each tile starts from is optionally written to the cache.
// Everything that does not need P (Q KV, the state update, the cache store) runs
// between the score phase and the barrier that publishes P, where the waves
// without a score block used to wait; V of the wave's columns stays in registers
// across it, so the next tile's stores need no barrier of their own: two a tile. With one workgroup per CU the
// walk is bound by this chain (one wave per SIMD): d=128, 16 heads x 1024 tokens in
// one segment 70.8 -> 61.6 us; the step of 4 x 32 heads x 16384 1780 -> 1752 us.
// ---------------------------------------------------------------------------
// NORM: every output row is divided by its root mean square (plus eps under the root) before it is
// stored, and the factor is written to rstd_out ([chain][token]) for the backward pass.
// WK, WV: elements per row of Q, K and of V, O in memory (<= D; see k_local).
// STATES: only the states are wanted (a backward pass that was given no state cache rebuilds it, Sec. 3.4's
// recomputation instead of caching): Q is not read, no scores and no outputs are computed; K, V are
// walked, every tile's entering state goes to the cache and the state is updated.
// ROLE kDq (float data): the walk over dO, V, K instead of Q, K, V, which produces dQ,
//     dQ_s = sum_{i<=s} lambda^(s-i) (do_s . v_i) k_i + lambda^s KV_in do_s,
// the same sums with the state transposed, a segment from each state the forward pass kept (WK, WV are then the
// widths of V and K). NORM: dO is dY and becomes dO on its way to LDS (NormTile). With a decay per token the row
// dots q.dq (q_rows: Q) go to rtok.
enum Role { kOutputs, kStates, kDq };
// LDS of the walk: row stride of the score tile (float: unpadded, so that two workgroups share a CU) and the
// staging area of the cache stores.
template <typename T, int CT>
constexpr int fwd_ldp() { return sizeof(T) == 4 ? CT : CT + WalkElem<T>::PAD; }
template <typename T, int D>
constexpr int fwd_stage() { return sizeof(T) == 4 ? 0 : D * 36; }
template <typename T, int CT, int D, bool TOKEN, bool RAGGED, bool NORM, int WK, int WV, Role ROLE, typename SH>
__global__ __launch_bounds__(D * 2, (sizeof(T) == 4 && D == 128 && ROLE == kDq && (TOKEN || NORM)) ? 1 : 2) void k_fwd(const T *__restrict__ Q, const T *__restrict__ K,
                                                const T *__restrict__ V, const float *__restrict__ decay,
                                                T *__restrict__ O, float *__restrict__ kv_out,
                                                T *__restrict__ cache, int cache_tiles, const float *__restrict__ scratch,
                                                const float *__restrict__ kv_in, const float *__restrict__ seglog, int carry,
                                                int H, int ntiles, int nseg, int tiles_per_seg, int ntok, int kvdiv,
                                                float *__restrict__ rstd_out, float eps, const T *__restrict__ yn,
                                                const float *__restrict__ rstd, const T *__restrict__ q_rows, float *__restrict__ rtok,
                                                float *__restrict__ kv_copy, SH sh) {
    using E = WalkElem<T>;
    constexpr bool STATES = ROLE == kStates, DQ = ROLE == kDq;
    constexpr int NT = D * 2, LDD = walk_ld<T, D>(), LDP = fwd_ldp<T, CT>(), DB = D / 32, NB = CT / 32, NKS = CT / E::KSTEP,
                  SPB = 32 / E::KSTEP, TILE = walk_tile<T>(CT, LDD);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t *sQ = (bf16_t *)smem;
    bf16_t *sK = sQ + TILE;
    bf16_t *sV = sK + TILE;
    bf16_t *sP = sV + TILE;
    bf16_t *sStage = sP + walk_tile<T>(CT, LDP);   // cache stores, bfloat16
    float *pw = (float *)(sStage + fwd_stage<T, D>());

    constexpr bool SHARED = is_shared<SH>, OWN = is_own<SH>;
    const int chain = blockIdx.y, seg = blockIdx.x, shard = SHARED ? blockIdx.z : 0, shards = SHARED ? gridDim.z : 1, nslots = shards * nseg;
    const int slot0 = shard * nseg + seg;   // among the segments of all sub-sequences of the launch
    const int t0 = seg * tiles_per_seg;
    const int t1 = min(t0 + tiles_per_seg, ntiles);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index, scalar
    Lane ln = fresh_lane();
    if constexpr (SHARED) {
        if (shard) {
            Q = at_shard(Q, sh.q, shard);
            K = at_shard(K, sh.k, shard);
            V = at_shard(V, sh.v, shard);
            O = at_shard(O, sh.out, shard);
            if constexpr (DQ) {
                if constexpr (NORM) {
                    yn = at_shard(yn, sh.yn, shard);
                    rstd = at_shard(rstd, sh.rstd, shard);
                }
                if (carry < 0) scratch = at_shard(scratch, sh.cache, shard);
            } else {
                kv_out = at_shard(kv_out, sh.kv_out, shard);
                cache = at_shard(cache, sh.cache, shard);
                if constexpr (NORM) rstd_out = at_shard(rstd_out, sh.rstd, shard);
            }
        }
    }
    // requests first (tile, then start state), table arithmetic while they fly
    K += kv_shift(chain, H, kvdiv, ntok, WK);   // K, V of this chain's K/V head
    V += kv_shift(chain, H, kvdiv, ntok, WV);
    auto koff = [&](int t) { return tile_off(chain, ntok, t, CT, WK); };
    auto voff = [&](int t) { return tile_off(chain, ntok, t, CT, WV); };
    // rows of tile `t` that exist: the last tile of a sub-sequence may be short
    auto nvalid = [&](int t) { return RAGGED ? min(CT, ntok - t * CT) : CT; };
    static_assert(!STATES || !NORM, "the states do not depend on the Norm");
    TileMover<T, CT, D, NT> mq, mk, mv;
    NormTile<T, CT, D, NT, WK> mn;   // kDq only
    const float *rstd_c = rstd + (size_t)chain * ntok;
    const float *lg = decay + (size_t)chain * ntok;  // per-token decay: `decay` is log g, [chain][token]
    typename TokenDecay<T, CT>::LogG lgreg = {};
    auto request_kv = [&](int t) __attribute__((always_inline)) {
        mk.template load_w<WK>(K + koff(t), nvalid(t));
        mv.template load_w<WV>(V + voff(t), nvalid(t));
        if constexpr (TOKEN) lgreg = TokenDecay<T, CT>::fetch(lg + (size_t)t * CT, nvalid(t));
    };
    auto request = [&](int t) __attribute__((always_inline)) {
        if constexpr (DQ && NORM) mn.load(yn + koff(t), rstd_c + (size_t)t * CT, nvalid(t));
        if constexpr (!STATES) mq.template load_w<WK>(Q + koff(t), nvalid(t));
        request_kv(t);
    };
    const int own = OWN && carry == kOwn ? t0 : 0;   // tiles before this segment that the workgroup takes the state through
    if (own) request_kv(0);
    else request(t0);
    f32x16 st[DB];
    {
        // kDq, carry < 0: the states are those that the forward pass kept, a buffer per sub-sequence
        const bool kept = DQ && carry == kKept;
        const float *states = scratch + (size_t)chain * (kept ? nseg : nslots) * WK * WV;
        auto load = [&](f32x16(&s)[DB], const float *g) {
            if constexpr (DQ) state_load_t_w<D, WV, WK>(ln, s, g, w);   // stored [d_k][d_v] = [WV][WK]
            else state_load_w<D, WK, WV>(ln, s, g, w);
        };
        if (carry > 0) {
            const Pieces pc(false, !OWN && carry == kCarriedPieces, shards, nseg, tiles_per_seg, ntiles);
            start_state<false, SHARED>(st, scratch + ((ptrdiff_t)chain * pc.slots - pc.base) * WK * WV, kv_in ? kv_in + (size_t)chain * WK * WV : nullptr,
                               SegDecay<TOKEN>(decay, seglog + ((ptrdiff_t)chain * pc.slots - pc.base), chain, H, pc.per_shard, pc.tiles * CT, ntok),
                               OWN && carry == kOwn ? 0 : piece_of<false>(pc, shard, seg), pc.per_shard, pc.per_shard * shards, WK * WV, load);
        } else load(st, states + (size_t)(kept ? seg : slot0) * WK * WV);
    }
    const auto dec = DecaySel<TOKEN, T, CT>::make(pw, decay, chain, H);
    typename E::frag vf[NKS];
    auto load_vf = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) vf[ks] = E::ld_ks(ln, sV, LDD, ks * E::KSTEP, 32 * w);
    };
    for (int t = 0; t < own; ++t) {   // the state alone (all of these tiles are whole)
        __syncthreads();
        mk.store(sK, LDD);
        mv.store(sV, LDD);
        if constexpr (TOKEN) dec.fill(lgreg);
        else if constexpr (E::PLANES == 3) dec.set_end(CT);   // float: weights rounded once, like the local pass's
        __syncthreads();
        if (t + 1 < own) request_kv(t + 1);
        else request(t0);
        ln = fresh_lane();
        const float lamC = dec.whole(CT);
        if constexpr (E::PLANES == 3) {
            unsigned lows = 0;
            auto weigh = [&](auto edge) __attribute__((always_inline)) {
                load_vf();
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) vf[ks] = dec.template weigh_after<false, decltype(edge)::value>(ln, vf[ks], ks, &lows);
            };
            weigh(std::false_type{});
            if (__builtin_expect(E::edge(lows), 0)) weigh(std::true_type{});
            decay_and_add<E, true>(ln, st, lamC, sK, LDD, vf);
        } else {
            load_vf();
#pragma unroll
            for (int ab = 0; ab < DB; ++ab) st[ab] *= lamC;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const typename E::frag vd = dec.template weigh_after<true>(ln, vf[ks], ks);
#pragma unroll
                for (int ab = 0; ab < DB; ++ab) st[ab] = E::mfma(E::ld_ks(ln, sK, LDD, ks * E::KSTEP, 32 * ab), vd, st[ab]);
            }
        }
    }
    if (own) __syncthreads();

    // State cache: the state KV_{t-1} that tile `t` starts from, rows a, columns c. bfloat16: every second tile, or every
    // tile (cache_tiles 2 or 1). Float: every cache_tiles-th, where the kDq walk starts; these are the segments' starts unless the caller chose the segments.
    [[maybe_unused]] int slot = 0;
    if constexpr (sizeof(T) == 4 && !DQ) {
        if (cache) slot = (t0 + cache_tiles - 1) / cache_tiles;   // the next to be written
    }
    auto to_cache = [&](int t) __attribute__((always_inline)) {
        if constexpr (sizeof(T) == 2) {
            const int half = cache_tiles - 1;
            if (cache && (t & half) == 0)
                cache_store<D, WK, WV>(ln, cache + ((size_t)chain * ((ntiles + half) >> half) + (t >> half)) * WK * WV, st, sStage + w * 32 * 36, w);
        } else if constexpr (!DQ) {
            if (cache && t == slot * cache_tiles) {
                const int slots = (ntiles + cache_tiles - 1) / cache_tiles;
                state_store_w<D, WK, WV>(ln, st, cache + ((size_t)chain * slots + slot++) * WK * WV, w);
            }
        }
    };
    to_cache(t0);
    if constexpr (E::PLANES == 3 && !STATES) {
        if (w == D / 32 - 1) clear_upper_scores<LDP>(ln, sP);
    }
    if (!DQ && kv_copy && slot0 == 0) state_store_w<D, WK, WV>(ln, st, kv_copy + (size_t)chain * WK * WV, w);
    if constexpr (RAGGED && !TOKEN) {
        __syncthreads();   // the power table
        dec.set_end(nvalid(t0));
    }

    for (int t = t0; t < t1; ++t) {
        // bfloat16: every wave is past the previous tile's second barrier, so Q, K, V and the tables are free; only P
        // may still be read. Float: V may be, too (its fragments are three times as large, too many to keep).
        if constexpr (E::PLANES == 3) __syncthreads();
        ln = fresh_lane();
        if constexpr (DQ && NORM) mn.apply(mq);
        if constexpr (!STATES) mq.store(sQ, LDD);
        mk.store(sK, LDD);
        mv.store(sV, LDD);
        if constexpr (TOKEN) dec.fill(lgreg);
        else if constexpr (RAGGED) {
            if (t > t0 && nvalid(t) < CT) dec.set_end(nvalid(t));
        }
        __syncthreads();
        if (t + 1 < t1) request(t + 1);
        // Output tiles are accumulated transposed: OT[c][i], c in this wave's column block.
        f32x16 acc[NB];
        if constexpr (!STATES) {
            // masked scores P (all waves share the lower-triangular blocks)
            masked_scores<T, CT, D, LDD, LDP, D / 32>(ln, sP, sK, sQ, dec, w);
#pragma unroll
            for (int ib = 0; ib < NB; ++ib) acc[ib] = f32x16{0};
            // inter: OT[c][i] = sum_a KV_{t-1}[a][c] Q[i][a], a taken in accumulator order
            if constexpr (E::PLANES == 1) {   // (float data: below)
#pragma unroll
                for (int ab = 0; ab < DB; ++ab)
#pragma unroll
                    for (int m = 0; m < E::NSUB; ++m) {
                        const typename E::frag sf = E::from_acc(st[ab], m);
#pragma unroll
                        for (int ib = 0; ib < NB; ++ib) acc[ib] = E::mfma(sf, E::ld_kp(ln, sQ, LDD, 32 * ib, 32 * ab, m), acc[ib]);
                    }
            }
            // Lambda: token r (1-based) carries lambda^r; the token is this lane's column
            if constexpr (E::PLANES == 1) {
#pragma unroll
                for (int ib = 0; ib < NB; ++ib) acc[ib] *= dec.upto(32 * ib + ln.r);
            }
        }
        // V of this wave's columns, for the state update and, behind the barrier, for P V
        ln = fresh_lane();
        // state update: KV <- lambda^CT KV + (diag{lambda^(CT-1-j)} K)^T V, weight applied to the V fragments
        const float lamC = dec.whole(nvalid(t));
        if constexpr (E::PLANES == 3) {
            unsigned lows = 0;
            auto inter_and_weigh = [&](auto edge) __attribute__((always_inline)) {
                constexpr bool EDGE = decltype(edge)::value;
                if constexpr (!STATES) {
                    static_assert(NB == 1, "one 32-token block per tile");
                    acc[0] = state_product<E, EDGE>(st, lows, [&](int i) { return E::ld_kp(ln, sQ, LDD, 0, 32 * (i / E::NSUB), i % E::NSUB); });
                    acc[0] *= dec.upto(ln.r);
                    ln = fresh_lane();
                }
                load_vf();
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) vf[ks] = dec.template weigh_after<!RAGGED, EDGE>(ln, vf[ks], ks, &lows);
            };
            inter_and_weigh(std::false_type{});
            if (__builtin_expect(E::edge(lows), 0)) inter_and_weigh(std::true_type{});
            decay_and_add<E>(ln, st, lamC, sK, LDD, vf);
        } else {
            load_vf();
#pragma unroll
            for (int ab = 0; ab < DB; ++ab) st[ab] *= lamC;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const typename E::frag vd = dec.template weigh_after<!RAGGED>(ln, vf[ks], ks);
#pragma unroll
                for (int ab = 0; ab < DB; ++ab) st[ab] = E::mfma(E::ld_ks(ln, sK, LDD, ks * E::KSTEP, 32 * ab), vd, st[ab]);
            }
        }
        if (t + 1 < t1) to_cache(t + 1);

        __syncthreads();  // P visible; Q, K, V and the tables consumed
        if constexpr (!STATES) {
            ln = fresh_lane();
            if constexpr (E::PLANES == 3) load_vf();
            // intra: OT[c][i] += sum_{j<=i} V[j][c] P[i][j]
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                for (int ib = ks / SPB; ib < NB; ++ib) acc[ib] = E::mfma(vf[ks], E::ld_kc(ln, sP, LDP, 32 * ib, ks * E::KSTEP), acc[ib]);
            if constexpr (DQ && TOKEN) {   // q.dq over this wave's 32 features, then over the waves
                float *red = pw + 3 * CT + 4;
#pragma unroll
                for (int ib = 0; ib < NB; ++ib) {
                    float s = 0.0f;
                    if (32 * w < WV && 32 * ib + ln.r < nvalid(t)) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 x = gload<f32x4>(q_rows + voff(t) + 32 * ib * WV + 32 * w + 8 * q, (ln.r * WV + 4 * ln.h) * sizeof(T));
#pragma unroll
                            for (int e = 0; e < 4; ++e) s += acc[ib][4 * q + e] * x[e];
                        }
                    }
                    s = add_other_half(s);
                    if (ln.h == 0) red[w * CT + 32 * ib + ln.r] = s;
                }
                __syncthreads();
                if ((int)threadIdx.x < nvalid(t)) {
                    float r = 0.0f;
#pragma unroll
                    for (int wv = 0; wv < D / 32; ++wv) r += red[wv * CT + threadIdx.x];
                    rtok[(size_t)chain * ntok + (size_t)t * CT + threadIdx.x] = r;
                }
            }
            if constexpr (NORM && !DQ) {
                // sum of squares of a token's row: this wave's 32 features, then the other waves' through LDS
                float *red = pw + 3 * CT + 4;
#pragma unroll
                for (int ib = 0; ib < NB; ++ib) {
                    float ss = 0.0f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) ss += acc[ib][i] * acc[ib][i];
                    ss = add_other_half(ss);
                    if (ln.h == 0) red[w * CT + 32 * ib + ln.r] = ss;
                }
                __syncthreads();
#pragma unroll
                for (int ib = 0; ib < NB; ++ib) {
                    float tot = 0.0f;
#pragma unroll
                    for (int wv = 0; wv < D / 32; ++wv) tot += red[wv * CT + 32 * ib + ln.r];
                    const float rs = rsqrtf(tot * (1.0f / WV) + eps);   // mean over the real value features (padding is zero)
                    acc[ib] *= rs;
                    if (w == 0 && ln.h == 0 && (!RAGGED || 32 * ib + ln.r < nvalid(t)))
                        rstd_out[(size_t)chain * ntok + (size_t)t * CT + 32 * ib + ln.r] = rs;
                }
            }
            T *o = O + voff(t);
#pragma unroll
            for (int ib = 0; ib < NB; ++ib) store_out_tile_t<T, D, WV>(ln, o, acc[ib], 32 * ib, w, nvalid(t));
        }
    }
    if (!DQ && seg == nseg - 1 && kv_out) state_store_w<D, WK, WV>(ln, st, kv_out + (size_t)chain * WK * WV, w);
}

// ---------------------------------------------------------------------------
// k_fwd8: k_fwd for bfloat16 at d = 128 in eight waves, one workgroup per CU. Two groups of four waves split the
// state by rows (a) and the output tile by token block:
//   group g holds KV[a in half g][c in w]: half the state update, half of Q KV for both token blocks;
//   the half of Q KV that belongs to the other group's token block goes through LDS (32 KB a tile), after which
//   group g finishes token block g: P V, Norm, store.
// Per wave and tile 16 - 30 matrix instructions instead of 38 - 46, half of the conversions and stores, and a second
// wave per SIMD to run while one waits. Bound by the traffic on whole tiles with one lambda per head (16 heads x 32768
// tokens, whole forward 172.9 -> 171.8 us); where every value fragment is weighted from a table, by that work, which
// the waves now share (ragged 179.1 -> 172.9, a decay per token 195.9 -> 180.2), as is Norm's (185.3 -> 179.5).
// ---------------------------------------------------------------------------
template <typename T, int CT, int D>
struct Fwd8Smem {
    static constexpr int LDD = walk_ld<T, D>(), LDP = CT + WalkElem<T>::PAD;
    static constexpr size_t P_OFF = 3 * (size_t)CT * LDD * sizeof(T);
    static constexpr size_t STAGE_OFF = P_OFF + (size_t)CT * LDP * sizeof(T);            // cache stores: 8 waves x 32 x 36
    static constexpr size_t X_OFF = STAGE_OFF + 8 * 32 * 36 * sizeof(T);                 // exchange: 8 waves x 32 x 32 float
    static constexpr size_t PW_OFF = X_OFF + 8 * 1024 * sizeof(float);
    static constexpr size_t TOTAL = PW_OFF + table_floats<CT>() * sizeof(float);
};
template <typename T, int CT, int D, bool TOKEN, bool RAGGED, bool NORM, Role ROLE, typename SH>
__global__ __launch_bounds__(D * 4) void k_fwd8(const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V,
                                                const float *__restrict__ decay, T *__restrict__ O, float *__restrict__ kv_out,
                                                T *__restrict__ cache, int cache_tiles, const float *__restrict__ scratch,
                                                const float *__restrict__ kv_in, const float *__restrict__ seglog, int carry, int H,
                                                int ntiles, int nseg, int tiles_per_seg, int ntok, int kvdiv,
                                                float *__restrict__ rstd_out, float eps, float *__restrict__ kv_copy, SH sh) {
    using E = WalkElem<T>;
    using F = typename E::frag;
    using SM = Fwd8Smem<T, CT, D>;
    static_assert(sizeof(T) == 2 && D == 128 && CT == 64, "two row halves, two token blocks");
    constexpr bool STATES = ROLE == kStates;
    constexpr int NT = D * 4, NW = D / 32, LDD = SM::LDD, LDP = SM::LDP, HB = D / 64, NB = CT / 32, NKS = CT / E::KSTEP, SPB = 32 / E::KSTEP;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    T *sQ = (T *)smem;
    T *sK = sQ + CT * LDD;
    T *sV = sK + CT * LDD;
    T *sP = (T *)(smem + SM::P_OFF);
    float *sX = (float *)(smem + SM::X_OFF);
    float *pw = (float *)(smem + SM::PW_OFF);

    constexpr bool SHARED = is_shared<SH>, OWN = is_own<SH>;
    const int chain = blockIdx.y, seg = blockIdx.x, shard = SHARED ? blockIdx.z : 0, shards = SHARED ? gridDim.z : 1, nslots = shards * nseg;
    const int slot0 = shard * nseg + seg;   // among the segments of all sub-sequences of the launch
    const int t0 = seg * tiles_per_seg;
    const int t1 = min(t0 + tiles_per_seg, ntiles);
    if constexpr (SHARED) {
        if (shard) {
            Q = at_shard(Q, sh.q, shard);
            K = at_shard(K, sh.k, shard);
            V = at_shard(V, sh.v, shard);
            O = at_shard(O, sh.out, shard);
            kv_out = at_shard(kv_out, sh.kv_out, shard);
            cache = at_shard(cache, sh.cache, shard);
            if constexpr (NORM) rstd_out = at_shard(rstd_out, sh.rstd, shard);
        }
    }
    const int w8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = w8 % NW, g = w8 / NW;   // value-feature block; row half of the state and token block of the output
    const int a0 = 64 * g;                // first state row of this wave
    T *stage = (T *)(smem + SM::STAGE_OFF) + w8 * 32 * 36;
    Lane ln = fresh_lane();
    K += kv_shift(chain, H, kvdiv, ntok, D);
    V += kv_shift(chain, H, kvdiv, ntok, D);
    auto off = [&](int t) { return tile_off(chain, ntok, t, CT, D); };
    auto nvalid = [&](int t) { return RAGGED ? min(CT, ntok - t * CT) : CT; };
    TileMover<T, CT, D, NT> mq, mk, mv;
    const float *lg = decay + (size_t)chain * ntok;
    typename TokenDecay<T, CT>::LogG lgreg = {};
    auto request_kv = [&](int t) __attribute__((always_inline)) {
        mk.load(K + off(t), nvalid(t));
        mv.load(V + off(t), nvalid(t));
        if constexpr (TOKEN) lgreg = TokenDecay<T, CT>::fetch(lg + (size_t)t * CT, nvalid(t));
    };
    auto request = [&](int t) __attribute__((always_inline)) {
        if constexpr (!STATES) mq.load(Q + off(t), nvalid(t));
        request_kv(t);
    };
    const int own = OWN && carry == kOwn ? t0 : 0;   // tiles before this segment that the workgroup takes the state through
    if (own) request_kv(0);
    else request(t0);
    f32x16 st[HB];   // st[ab][i] = KV[a0 + 32 ab + acc_row(i)][32 w + r]
    {
        const float *states = scratch + (size_t)chain * nslots * D * D;
        auto load = [&](f32x16(&s)[HB], const float *p) { state_load_w<D, D, D, HB>(ln, s, p + a0 * D, w); };
        if (carry) {
            const Pieces pc(false, !OWN && carry == kCarriedPieces, shards, nseg, tiles_per_seg, ntiles);
            start_state<false, SHARED>(st, scratch + ((ptrdiff_t)chain * pc.slots - pc.base) * D * D, kv_in ? kv_in + (size_t)chain * D * D : nullptr,
                               SegDecay<TOKEN>(decay, seglog + ((ptrdiff_t)chain * pc.slots - pc.base), chain, H, pc.per_shard, pc.tiles * CT, ntok),
                               OWN && carry == kOwn ? 0 : piece_of<false>(pc, shard, seg), pc.per_shard, pc.per_shard * shards, D * D, load);
        } else load(st, states + (size_t)slot0 * D * D);
    }
    const auto dec = DecaySel<TOKEN, T, CT>::make(pw, decay, chain, H);
    for (int t = 0; t < own; ++t) {   // the state alone (all of these tiles are whole)
        __syncthreads();
        mk.store(sK, LDD);
        mv.store(sV, LDD);
        if constexpr (TOKEN) dec.fill(lgreg);
        __syncthreads();
        if (t + 1 < own) request_kv(t + 1);
        else request(t0);
        ln = fresh_lane();
        const float lamC = dec.whole(CT);
#pragma unroll
        for (int ab = 0; ab < HB; ++ab) st[ab] *= lamC;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            const F vd = dec.template weigh_after<true>(ln, E::ld_ks(ln, sV, LDD, ks * E::KSTEP, 32 * w), ks);
#pragma unroll
            for (int ab = 0; ab < HB; ++ab) st[ab] = E::mfma(E::ld_ks(ln, sK, LDD, ks * E::KSTEP, a0 + 32 * ab), vd, st[ab]);
        }
    }
    if (own) __syncthreads();
    auto to_cache = [&](int t) __attribute__((always_inline)) {
        const int half = cache_tiles - 1;
        if (cache && (t & half) == 0)
            cache_store<D, D, D, HB>(ln, cache + ((size_t)chain * ((ntiles + half) >> half) + (t >> half)) * D * D + a0 * D, st, stage, w);
    };
    to_cache(t0);
    if (kv_copy && slot0 == 0) state_store_w<D, D, D, HB>(ln, st, kv_copy + (size_t)chain * D * D + a0 * D, w);
    if constexpr (RAGGED && !TOKEN) {
        __syncthreads();   // the power table
        dec.set_end(nvalid(t0));
    }

    for (int t = t0; t < t1; ++t) {
        // Every wave is past the previous tile's second barrier: only P, the exchange and (Norm) the row sums may still
        // be read, and those are written behind the next barrier.
        ln = fresh_lane();
        if constexpr (!STATES) mq.store(sQ, LDD);
        mk.store(sK, LDD);
        mv.store(sV, LDD);
        if constexpr (TOKEN) dec.fill(lgreg);
        else if constexpr (RAGGED) {
            if (t > t0 && nvalid(t) < CT) dec.set_end(nvalid(t));
        }
        __syncthreads();
        if (t + 1 < t1) request(t + 1);
        f32x16 part = {0};   // OT[c][i], c in w, i in token block g
        if constexpr (!STATES) {
            masked_scores<T, CT, D, LDD, LDP, 2 * NW>(ln, sP, sK, sQ, dec, w8);
            // this row half's share of Q KV, both token blocks
            f32x16 acc[NB];
#pragma unroll
            for (int ib = 0; ib < NB; ++ib) acc[ib] = f32x16{0};
#pragma unroll
            for (int ab = 0; ab < HB; ++ab)
#pragma unroll
                for (int m = 0; m < E::NSUB; ++m) {
                    const F sf = E::from_acc(st[ab], m);
#pragma unroll
                    for (int ib = 0; ib < NB; ++ib) acc[ib] = E::mfma(sf, E::ld_kp(ln, sQ, LDD, 32 * ib, a0 + 32 * ab, m), acc[ib]);
                }
            // the other group's block to LDS, lane-contiguous
            const f32x16 give = g ? acc[0] : acc[1];
            part = g ? acc[1] : acc[0];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4 *)(sX + (w8 * 4 + q) * 256 + 4 * ln.id) = f32x4{give[4 * q], give[4 * q + 1], give[4 * q + 2], give[4 * q + 3]};
        }
        const float up = STATES ? 0.0f : dec.upto(32 * g + ln.r);
        ln = fresh_lane();
        F vf[NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) vf[ks] = E::ld_ks(ln, sV, LDD, ks * E::KSTEP, 32 * w);
        const float lamC = dec.whole(nvalid(t));
#pragma unroll
        for (int ab = 0; ab < HB; ++ab) st[ab] *= lamC;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            const F vd = dec.template weigh_after<!RAGGED>(ln, vf[ks], ks);
#pragma unroll
            for (int ab = 0; ab < HB; ++ab) st[ab] = E::mfma(E::ld_ks(ln, sK, LDD, ks * E::KSTEP, a0 + 32 * ab), vd, st[ab]);
        }
        if (t + 1 < t1) to_cache(t + 1);

        __syncthreads();  // P and the exchange visible; Q, K, V and the tables consumed
        if constexpr (!STATES) {
            ln = fresh_lane();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 x = *(const f32x4 *)(sX + (((1 - g) * NW + w) * 4 + q) * 256 + 4 * ln.id);
#pragma unroll
                for (int e = 0; e < 4; ++e) part[4 * q + e] += x[e];
            }
            part *= up;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
                if (g == 1 || ks < SPB) part = E::mfma(vf[ks], E::ld_kc(ln, sP, LDP, 32 * g, ks * E::KSTEP), part);
            if constexpr (NORM) {
                float *red = pw + 3 * CT + 4;
                float ss = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; ++i) ss += part[i] * part[i];
                ss = add_other_half(ss);
                if (ln.h == 0) red[w * CT + 32 * g + ln.r] = ss;
                __syncthreads();
                float tot = 0.0f;
#pragma unroll
                for (int wv = 0; wv < NW; ++wv) tot += red[wv * CT + 32 * g + ln.r];
                const float rs = rsqrtf(tot * (1.0f / D) + eps);
                part *= rs;
                if (w == 0 && ln.h == 0 && (!RAGGED || 32 * g + ln.r < nvalid(t)))
                    rstd_out[(size_t)chain * ntok + (size_t)t * CT + 32 * g + ln.r] = rs;
            }
            store_out_tile_t<T, D>(ln, O + off(t), part, 32 * g, w, nvalid(t));
        }
    }
    if (seg == nseg - 1 && kv_out) state_store_w<D, D, D, HB>(ln, st, kv_out + (size_t)chain * D * D + a0 * D, w);
}

// ---------------------------------------------------------------------------
// Backward walks, one segment of one head, tiles descending (Alg. 3 per tile):
//   dSm = (dO V^T) (.) M,  Sm = (Q K^T) (.) M
//   dQ  = dSm K + Lambda (dO KV_{t-1}^T)
//   dK  = dSm^T Q + (lambda^CT Lambda^-1) (V dKV^T)
//   dV  = Sm^T dO + (lambda^CT Lambda^-1) (K dKV)
//   dKV <- lambda^CT dKV + (Lambda Q)^T dO
// dKV is the state received from the right (gradient w.r.t. KV_t).
//
// k_bwdkv (float data) produces dK, dV and the dKV update only; dQ, which needs no
// dKV but the forward states, is a forward walk of its own (k_fwd, kDq) from one
// kept state per automatic segment. A float state per 32-token tile would be as many
// bytes as Q, K, V and O together, written by the forward pass and read here (268 MB
// each way at 16 heads x 8192 tokens, d=128; that step, 682 us with such a cache and
// fp32 matrix instructions, takes 469 with this, the operand split of WalkElem and 512
// forward workgroups). Both walks are bound by the split's vector instructions and the
// matrix instructions, which a wave issues one after the other (about 1300 and 120 a tile).
// Workgroups of 2 * D/32 waves. Two groups of waves keep dKV in registers in the
// orientation their product needs, so nothing is exchanged:
//   group 0 holds dKV[a][c in w] (rows a) and produces dV (dV_inter contracts a),
//   group 1 holds dKV[a in w][c] (rows c) and produces dK (dK_inter contracts c);
// under the exchange K<->V, Q<->dO, S<->dS the two are the same code. The products
// that do not need the scores run before the barrier that publishes them, where the
// waves without a score block would wait.
// NORM: dO is dY, the gradient w.r.t. the normalised output `yn`; every dY tile is turned into dO on its
// way to LDS (NormTile) from `yn` and `rstd` ([chain][token]).
// WK, WV: elements per row of Q, K, dK and of V, dO, dV in memory (<= D; see k_local).
// TOKEN: rtok holds q.dq on entry and q.dq - k.dk on exit.
// ---------------------------------------------------------------------------
template <typename T, int CT, int D>
struct BwdkvSmem {
    static constexpr int LDD = walk_ld<T, D>(), LDP = CT + WalkElem<T>::PAD;
    static constexpr int TILE = walk_tile<T>(CT, LDD), PTILE = walk_tile<T>(CT, LDP);   // elements
    static constexpr size_t PW_OFF = (4 * (size_t)TILE + 2 * PTILE) * sizeof(bf16_t);
    static constexpr size_t TOTAL = PW_OFF + table_floats<CT>() * sizeof(float);
};

template <typename T, int CT, int D, bool TOKEN, bool RAGGED, bool NORM, int WK, int WV, typename SH>
__global__ __launch_bounds__(D * 4) void k_bwdkv(const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V,
                                                 const T *__restrict__ dO, const float *__restrict__ decay, T *__restrict__ dK,
                                                 T *__restrict__ dV, float *__restrict__ dkv_in, const float *__restrict__ scratch,
                                                 const float *__restrict__ dkv_out, const float *__restrict__ seglog, int carry,
                                                 float *__restrict__ rtok, int H, int ntiles, int nseg, int tiles_per_seg,
                                                 int ntok, int kvdiv, const T *__restrict__ yn, const float *__restrict__ rstd,
                                                 float *__restrict__ dkv_copy, SH sh) {
    using E = WalkElem<T>;
    using F = typename E::frag;
    using SM = BwdkvSmem<T, CT, D>;
    static_assert(CT == 32, "one 32-token block per tile");
    constexpr int NT = D * 4, NW = D / 32, LDD = SM::LDD, LDP = SM::LDP, DB = D / 32, NKS = CT / E::KSTEP;
    constexpr int KB = WK / 32, VB = WV / 32;   // real 32-wide feature blocks of the key and value side
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t *sV = (bf16_t *)smem;
    bf16_t *sdO = sV + SM::TILE;
    bf16_t *sK = sdO + SM::TILE;
    bf16_t *sQ = sK + SM::TILE;
    bf16_t *sS = sQ + SM::TILE;
    bf16_t *sDS = sS + SM::PTILE;
    float *pw = (float *)(smem + SM::PW_OFF);

    constexpr bool SHARED = is_shared<SH>, OWN = is_own<SH>;
    const int chain = blockIdx.y, seg = blockIdx.x, shard = SHARED ? blockIdx.z : 0, shards = SHARED ? gridDim.z : 1, nslots = shards * nseg;
    const int slot0 = shard * nseg + seg;   // among the segments of all sub-sequences of the launch
    const int t0 = seg * tiles_per_seg;
    const int t1 = min(t0 + tiles_per_seg, ntiles);
    if constexpr (SHARED) {
        if (shard) {
            Q = at_shard(Q, sh.q, shard);
            K = at_shard(K, sh.k, shard);
            V = at_shard(V, sh.v, shard);
            dO = at_shard(dO, sh.dout, shard);
            dK = at_shard(dK, sh.dk, shard);
            dV = at_shard(dV, sh.dv, shard);
            dkv_in = at_shard(dkv_in, sh.dkv_in, shard);
            if constexpr (NORM) {
                yn = at_shard(yn, sh.yn, shard);
                rstd = at_shard(rstd, sh.rstd, shard);
            }
        }
    }
    const int w8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = w8 % NW;    // feature block of this wave's output
    const int rg = w8 / NW;   // group: 0 produces dV, 1 produces dK
    const bool own_block = rg ? w < KB : w < VB;   // (dimensions that differ: the block is not padding)
    Lane ln = fresh_lane();
    // rows of tile `t` that exist: only the first tile walked, the sub-sequence's last, may be short
    auto nvalid = [&](int t) { return RAGGED ? min(CT, ntok - t * CT) : CT; };
    K += kv_shift(chain, H, kvdiv, ntok, WK);   // K, V of this chain's K/V head
    V += kv_shift(chain, H, kvdiv, ntok, WV);
    auto koff = [&](int t) { return tile_off(chain, ntok, t, CT, WK); };
    auto voff = [&](int t) { return tile_off(chain, ntok, t, CT, WV); };

    TileMover<T, CT, D, NT> mv, mo, mk, mq;
    NormTile<T, CT, D, NT, WV> mn;
    const float *rstd_c = rstd + (size_t)chain * ntok;
    const float *lg = decay + (size_t)chain * ntok;  // per-token decay: `decay` is log g, [chain][token]
    typename TokenDecay<T, CT>::LogG lgreg = {};
    auto request = [&](int t, int n) __attribute__((always_inline)) {
        mv.template load_w<WV>(V + voff(t), n);
        mo.template load_w<WV>(dO + voff(t), n);
        mk.template load_w<WK>(K + koff(t), n);
        mq.template load_w<WK>(Q + koff(t), n);
        if constexpr (NORM) mn.load(yn + voff(t), rstd_c + (size_t)t * CT, n);
        if constexpr (TOKEN) lgreg = TokenDecay<T, CT>::fetch(lg + (size_t)t * CT, n);
    };
    // what the state alone needs, of the tiles behind this segment that the workgroup takes it through
    auto request_qdo = [&](int t) __attribute__((always_inline)) {
        mo.template load_w<WV>(dO + voff(t), nvalid(t));
        mq.template load_w<WK>(Q + koff(t), nvalid(t));
        if constexpr (NORM) mn.load(yn + voff(t), rstd_c + (size_t)t * CT, nvalid(t));
        if constexpr (TOKEN) lgreg = TokenDecay<T, CT>::fetch(lg + (size_t)t * CT, nvalid(t));
    };
    const int own = OWN && carry == kOwn ? ntiles - t1 : 0;   // tiles behind this segment that the workgroup takes the state through
    if (own) request_qdo(ntiles - 1);
    else request(t1 - 1, nvalid(t1 - 1));
    const auto dec = DecaySel<TOKEN, T, CT>::make(pw, decay, chain, H);
    float *rs = pw + 3 * CT + 4;   // one row of k.dk sums per wave of group 1
    auto flush_r = [&](int tile) {
        if ((int)threadIdx.x < nvalid(tile)) {
            float r = 0.0f;
#pragma unroll
            for (int wv = 0; wv < NW; ++wv) r += rs[wv * CT + threadIdx.x];
            rtok[(size_t)chain * ntok + (size_t)tile * CT + threadIdx.x] -= r;
        }
    };

    const bf16_t *sX1 = rg ? sV : sK;     // inter operand: token rows, features contracted with the state
    const bf16_t *sX2 = rg ? sQ : sdO;    // intra operand and state-update B operand: [token][feature in w]
    const bf16_t *sUA = rg ? sdO : sQ;    // state-update A operand: [token][feature of the state rows]
    const bf16_t *sPm = rg ? sDS : sS;    // masked score tile P[i][j] of this product

    // st[blk][i]: group 0: dKV[32 blk + acc_row(i)][32 w + r]; group 1: dKV[32 w + r][32 blk + acc_row(i)]
    f32x16 st[DB];
    {
        const float *states = scratch + (size_t)chain * nslots * WK * WV;
        auto load = [&](f32x16(&s)[DB], const float *g) {
            if (rg == 0) state_load_w<D, WK, WV>(ln, s, g, w);
            else state_load_t_w<D, WK, WV>(ln, s, g, w);
        };
        if (carry) {
            const Pieces pc(true, !OWN && carry == kCarriedPieces, shards, nseg, tiles_per_seg, ntiles);
            start_state<true, SHARED>(st, scratch + ((ptrdiff_t)chain * pc.slots - pc.base) * WK * WV, dkv_out ? dkv_out + (size_t)chain * WK * WV : nullptr,
                              SegDecay<TOKEN>(decay, seglog + ((ptrdiff_t)chain * pc.slots - pc.base), chain, H, pc.per_shard, pc.tiles * CT, ntok),
                              OWN && carry == kOwn ? pc.per_shard * shards - 1 : piece_of<true>(pc, shard, seg), pc.per_shard, pc.per_shard * shards, WK * WV, load);
        } else load(st, states + (size_t)slot0 * WK * WV);
        if (dkv_copy && slot0 == nslots - 1 && rg == 0) state_store_w<D, WK, WV>(ln, st, dkv_copy + (size_t)chain * WK * WV, w);
    }
    for (int t = ntiles - 1; t >= ntiles - own; --t) {
        __syncthreads();
        if constexpr (NORM) mn.apply(mo);
        mo.store(sdO, LDD);
        mq.store(sQ, LDD);
        if constexpr (TOKEN) dec.fill(lgreg);
        __syncthreads();
        if (t > t1) request_qdo(t - 1);
        else request(t1 - 1, CT);
        ln = fresh_lane();
        if (own_block) {
            F x2[NKS];
            unsigned lows = 0;
            auto weigh = [&](auto edge) __attribute__((always_inline)) {
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks)
                    x2[ks] = dec.template weigh_upto_once<decltype(edge)::value>(ln, E::ld_ks(ln, sX2, LDD, ks * E::KSTEP, 32 * w), ks, &lows);
            };
            weigh(std::false_type{});
            if (__builtin_expect(E::edge(lows), 0)) weigh(std::true_type{});
            decay_and_add<E, true>(ln, st, dec.whole(nvalid(t)), sUA, LDD, x2);
        }
    }

    if (w8 < 2) clear_upper_scores<LDP>(ln, w8 ? sDS : sS);
    for (int t = t1 - 1; t >= t0; --t) {
        __syncthreads();  // previous tile fully consumed
        ln = fresh_lane();
        if constexpr (NORM) mn.apply(mo);
        mv.store(sV, LDD);
        mo.store(sdO, LDD);
        mk.store(sK, LDD);
        mq.store(sQ, LDD);
        if constexpr (TOKEN) dec.fill(lgreg);
        __syncthreads();
        ln = fresh_lane();
        if constexpr (TOKEN) {
            if (t < t1 - 1) flush_r(t + 1);
        }
        if (t > t0) request(t - 1, CT);
        // masked scores S^T = K Q^T and dS^T = V dO^T (over the real key and value features), a 16x16 block at a time
        for (int blk = w8; blk < 2 * kScoreBlocks16; blk += 2 * NW) {
            const int b = blk % kScoreBlocks16, jb = score_jb16(b), ib = score_ib16(b);
            if (blk < kScoreBlocks16) score_block16<LDD, LDP, WK>(ln, sS, sK, sQ, jb, ib, dec);
            else score_block16<LDD, LDP, WV>(ln, sDS, sV, sdO, jb, ib, dec);
        }
        ln = fresh_lane();

        const int nv = nvalid(t);
        f32x16 acc = {0};   // dV^T[c in w][j] (group 0) or dK^T[a in w][j] (group 1)
        F x2[NKS];
        auto load_x2 = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) x2[ks] = E::ld_ks(ln, sX2, LDD, ks * E::KSTEP, 32 * w);
        };
        if (own_block) {
            unsigned lows = 0;
            auto inter_and_weigh = [&](auto edge) __attribute__((always_inline)) {
                constexpr bool EDGE = decltype(edge)::value;
                acc = state_product<E, EDGE>(st, lows, [&](int i) { return E::ld_kp(ln, sX1, LDD, 0, 32 * (i / E::NSUB), i % E::NSUB); });
                acc *= dec.after(ln.r, nv);
                load_x2();
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) x2[ks] = dec.template weigh_upto<EDGE>(ln, x2[ks], ks, &lows);
            };
            inter_and_weigh(std::false_type{});
            if (__builtin_expect(E::edge(lows), 0)) inter_and_weigh(std::true_type{});
            // dKV <- lambda^CT dKV + (Lambda Q)^T dO, in this group's orientation
            decay_and_add<E>(ln, st, dec.whole(nv), sUA, LDD, x2);
        }
        __syncthreads();  // scores visible
        ln = fresh_lane();
        if (own_block) {
            load_x2();
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) acc = E::mfma(x2[ks], E::ld_ks(ln, sPm, LDP, ks * E::KSTEP, 0), acc);
            if (rg) store_out_tile_t<T, D, WK>(ln, dK + koff(t), acc, 0, w, nv);
            else store_out_tile_t<T, D, WV>(ln, dV + voff(t), acc, 0, w, nv);
        }
        if constexpr (TOKEN) {
            if (rg == 1) {
                const float s = own_block ? rowdot<T>(ln, acc, sK, LDD, 0, w) : 0.0f;
                if (ln.h == 0) rs[w * CT + ln.r] = s;
            }
        }
    }
    if constexpr (TOKEN) {
        __syncthreads();
        flush_r(t0);
    }
    if (seg == 0 && rg == 0) state_store_w<D, WK, WV>(ln, st, dkv_in + (size_t)chain * WK * WV, w);
}

// ---------------------------------------------------------------------------
// k_bwd8p: the backward walk for bfloat16 tiles of 64 tokens, one workgroup of
// 2 * D/32 waves per CU:
//   - every input tile, the masked score tiles and the cached state live in LDS
//     at once;
//   - the waves form two groups that each keep dKV in registers in the
//     orientation their product needs, so nothing is exchanged:
//       group 0 holds dKV[a][c in w] (rows a) and produces dV (dV_inter contracts a),
//       group 1 holds dKV[a in w][c] (rows c) and produces dK (dK_inter contracts c);
//     under the exchange K<->V, Q<->dO, S<->dS the two products are the same
//     code, including the dKV update, so the groups differ only in pointers;
//   - dQ needs only the cached state and is split by token block between them
//     (group 0, which the hardware favours when both wait to issue, takes the
//     block with the longer key range);
//   - the state cache holds one state per PAIR of tiles (half the cache traffic
//     of both passes). Tiles are walked in reverse as pairs (E = even tile, O =
//     the odd tile after it) and the cache gives KV at the start of E. The O
//     tile's dQ needs the state one tile later,
//         KV_mid = lambda^CT KV + (diag{lambda^(CT-1-j)} K_E)^T V_E   (state update of Sec. 3.2);
//     instead of rebuilding it, dQ of the O tile treats the pair as one chunk of 2 CT
//     tokens (Alg. 3 with C = 2 CT, restricted to the rows of the O tile):
//         dQ_O = Lambda' dO_O KV^T + [(dO_O V_E^T) (.) M'] K_E + [(dO_O V_O^T) (.) M] K_O,
//     Lambda'_i = lambda^(CT+i), M'_ij = lambda^(CT+i-j): one more masked score tile
//     (sDX) and four more contraction steps, and the cached tile stays in LDS for
//     both tiles. K_E, V_E are needed for the E tile anyway and are simply fetched
//     one tile early. Per pair: six barriers, 9 tile loads, one cache-tile load.
// An odd tile count leaves the last pair without its O tile: nothing of it is
// read, its phase is skipped and the E tile is the one that may be short.
// kTiles: the cache holds every tile's state (cache_every_tile), the tiles are
// walked one by one, each as an E tile: four input tiles in LDS, three barriers.
// kHalves: a state per pair, but a workgroup takes one tile of it, as E or as O tile
// (short sequences, whose few workgroups leave CUs idle and are bound by the length
// of a workgroup's chain: 16 heads x 256 tokens, step 38.0 -> 24.9 us together with
// the start states computed by the workgroups). One copy of the products in either
// role, so that less code is fetched for a single tile.
// ---------------------------------------------------------------------------
// (Bounds of two waves per SIMD: with one, the compiler holds the accumulators of d = 64 in the other half of the register file and
// every value takes a move to get at, a third of the vector instructions. Steps, d=64: bf16 16 heads x 128 tokens 18.3 -> 17.3
// us, x 512 29.2 -> 27.2, x 8192 83.6 -> 81.6, 2 x 32768 95 -> 92. k_bwdkv gains nothing by it.)
enum BwdWalk { kPairs, kTiles, kHalves };
template <typename T, int CT, int D, BwdWalk MODE = kPairs>
struct Bwd8pSmem {
    static constexpr bool BY_TILES = MODE == kTiles;
    // d = 64, in pairs: of the score tiles only the 32x32 blocks on and below the diagonal, and all four of the cross tile; the
    // cached state in registers (each wave reads its own rows only). The space (108 -> 79 KB) lets a second workgroup onto the
    // CU, which runs while one waits at a barrier: steps 16 heads x 32768 tokens 257 -> 237 us, 32 x 8192 136 -> 126, 128 x 2048
    // 127 -> 115. (Unpadded rows of 64 elements in swizzled order instead of 72: 15 % more vector instructions, 5 % slower.)
    static constexpr bool BLOCKS = D == 64 && MODE == kPairs;
    static constexpr int LDD = BLOCKS ? 72 : walk_ld<T, D>(), LDP = BLOCKS ? kBlockLd : CT + WalkElem<T>::PAD;
    static constexpr size_t TILE = (size_t)CT * LDD * sizeof(T);
    static constexpr int P_ELEMS = BLOCKS ? 3 * 1024 : CT * LDP, X_ELEMS = BY_TILES ? 0 : BLOCKS ? 4 * 1024 : CT * LDP;
    static constexpr size_t P_OFF = (BY_TILES ? 4 : 6) * TILE;
    static constexpr size_t C_OFF = P_OFF + (2 * (size_t)P_ELEMS + X_ELEMS) * sizeof(T);   // S, dS and the cross tile dS(O x E)
    // block of keys jb at queries ib
    static DEVI T *block(T *tile, int ib, int jb) { return tile + (BLOCKS ? 1024 * (ib ? 1 + jb : 3 * jb) : 32 * ib * LDP + 32 * jb); }
    static constexpr size_t PW_OFF = C_OFF + (BLOCKS ? 0 : (size_t)D * LDD * sizeof(T));
    // decay tables of the O tile and of the E tile, then one row of per-token partial sums per wave
    static constexpr int TABLES = (BY_TILES ? 1 : 2) * 3 * CT;
    static constexpr size_t TOTAL = PW_OFF + (TABLES + 4 + D / 16 * CT) * sizeof(float);
};

// WK, WV: elements per row of Q, K, dQ, dK and of V, dO, dV in memory (<= D; see k_local).
template <typename T, int CT, int D, bool TOKEN, bool RAGGED, bool NORM, int WK, int WV, BwdWalk MODE, typename SH>
__global__ __launch_bounds__(D * 4, 2) void k_bwd8p(const T *__restrict__ Q, const T *__restrict__ K,
                                                  const T *__restrict__ V, const T *__restrict__ dO,
                                                  const float *__restrict__ decay, const T *__restrict__ cache,
                                                  T *__restrict__ dQ, T *__restrict__ dK, T *__restrict__ dV,
                                                  float *__restrict__ dkv_in, const float *__restrict__ scratch,
                                                  const float *__restrict__ dkv_out, const float *__restrict__ seglog, int carry,
                                                  float *__restrict__ rtok,
                                                  int H, int ntiles, int nseg, int tiles_per_seg, int ntok, int kvdiv,
                                                  const T *__restrict__ yn, const float *__restrict__ rstd, float *__restrict__ dkv_copy,
                                                  SH sh) {
    using E = WalkElem<T>;
    using F = typename E::frag;
    constexpr bool BY_TILES = MODE == kTiles, HALVES = MODE == kHalves;
    using SM = Bwd8pSmem<T, CT, D, MODE>;
    static_assert(CT == 64, "two 32-token blocks per tile");
    static_assert(!is_own<SH> || MODE != kPairs, "in pairs: from states in the scratch");
    static_assert(RAGGED || MODE == kPairs, "one by one: one instance for any number of tiles and any length of the last");
    constexpr int NT = D * 4, NW = D / 32, LDD = SM::LDD, LDP = SM::LDP, DB = D / 32, NB = CT / 32, NKS = CT / E::KSTEP,
                  NKD = D / E::KSTEP, SPB = 32 / E::KSTEP;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    T *sVO = (T *)smem;            // V of the O tile
    T *sdO = sVO + CT * LDD;       // dO of the tile being processed
    T *sKO = sdO + CT * LDD;       // K of the O tile
    T *sQ = sKO + CT * LDD;        // Q of the tile being processed
    T *sVE = BY_TILES ? sVO : sQ + CT * LDD;    // V of the E tile
    T *sKE = BY_TILES ? sKO : sVE + CT * LDD;   // K of the E tile
    T *sS = (T *)(smem + SM::P_OFF);
    T *sDS = sS + SM::P_ELEMS;
    T *sDX = sDS + SM::P_ELEMS;    // masked dS between the O tile's queries and the E tile's keys
    T *sC = (T *)(smem + SM::C_OFF);
    float *pw = (float *)(smem + SM::PW_OFF);

    constexpr bool SHARED = is_shared<SH>, OWN = is_own<SH>;
    const int chain = blockIdx.y, seg = blockIdx.x, shard = SHARED ? blockIdx.z : 0, shards = SHARED ? gridDim.z : 1, nslots = shards * nseg;
    const int slot0 = shard * nseg + seg;   // among the segments of all sub-sequences of the launch
    if constexpr (SHARED) {
        if (shard) {
            Q = at_shard(Q, sh.q, shard);
            K = at_shard(K, sh.k, shard);
            V = at_shard(V, sh.v, shard);
            dO = at_shard(dO, sh.dout, shard);
            dK = at_shard(dK, sh.dk, shard);
            dV = at_shard(dV, sh.dv, shard);
            dkv_in = at_shard(dkv_in, sh.dkv_in, shard);
            if constexpr (NORM) {
                yn = at_shard(yn, sh.yn, shard);
                rstd = at_shard(rstd, sh.rstd, shard);
            }
            dQ = at_shard(dQ, sh.dq, shard);
            cache = at_shard(cache, sh.cache, shard);
        }
    }
    const int t0 = seg * tiles_per_seg;                                  // pairs: even
    // even: the last pair may lack its O tile
    const int t1 = MODE != kPairs ? min(t0 + tiles_per_seg, ntiles) : (min(t0 + tiles_per_seg, ntiles) + (RAGGED ? 1 : 0)) & ~1;
    auto nvalid = [&](int t) { return RAGGED ? max(min(CT, ntok - t * CT), 0) : CT; };  // rows of tile `t` that exist
    const int w8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = w8 % NW;    // feature block of this wave's outputs
    const int rg = w8 / NW;   // group: 0 produces dV, 1 produces dK
    Lane ln = fresh_lane();

    K += kv_shift(chain, H, kvdiv, ntok, WK);   // K, V of this chain's K/V head
    V += kv_shift(chain, H, kvdiv, ntok, WV);
    auto koff = [&](int t) { return tile_off(chain, ntok, t, CT, WK); };
    auto voff = [&](int t) { return tile_off(chain, ntok, t, CT, WV); };
    TileMover<T, CT, D, NT> mvO, moX, mkO, mqX, mvE, mkE;   // moX / mqX carry dO, Q of the O tile, then of the E tile
    TileMover<T, D, D, NT> mc;                               // cached state at the start of the E tile
    constexpr bool C_REGS = SM::BLOCKS;                      // (or its fragments: the tile's in use, and the next)
    F cf[C_REGS ? NKD : 1], cnext[C_REGS ? NKD : 1];
    const T *ctile = cache + (size_t)chain * (BY_TILES ? ntiles : (ntiles + 1) / 2) * WK * WV;   // [WK][WV] per slot
    // With a decay per token (`decay` = log g, [chain][token]) the O and the E tile have their own
    // tables; with one lambda per head both names refer to the same table.
    const auto decO = DecaySel<TOKEN, T, CT>::make(pw, decay, chain, H);
    const auto decE = [&] {
        if constexpr (TOKEN && !BY_TILES) return TokenDecay<T, CT>(pw + 3 * CT);
        else return decO;
    }();
    // weight key j of the E tile carries at query i of the O tile, and the E tile's entering state at query i
    // (one lambda per head: powers CT+1 .. 2 CT of the same table)
    auto cross_weight = [&](int i, int j) {
        if constexpr (TOKEN) return decO.upto(i) * decE.after(j, CT);
        else return decO.pw[CT + i - j];
    };
    auto far_upto = [&](int i) {
        if constexpr (TOKEN) return decO.upto(i) * decE.whole(CT);
        else return decO.pw[CT + i + 1];
    };
    const float *lg = decay + (size_t)chain * ntok;
    typename TokenDecay<T, CT>::LogG lgO = {}, lgE = {};
    // per-token decay: r_t = q_t.dq_t - k_t.dk_t, one partial row per wave, summed and written per tile
    float *rs = pw + SM::TABLES + 4;
    auto flush_r = [&](int tile) {
        if (threadIdx.x < CT) {
            float r = 0.0f;
#pragma unroll
            for (int wv = 0; wv < 2 * NW; ++wv) r += rs[wv * CT + threadIdx.x];
            if (!RAGGED || tile * CT + (int)threadIdx.x < ntok) rtok[(size_t)chain * ntok + (size_t)tile * CT + threadIdx.x] = r;
        }
    };
    NormTile<T, CT, D, NT, WV> mnX;  // NORM: partner of moX (dO is dY; see NormTile)
    const float *rstd_c = rstd + (size_t)chain * ntok;
    auto load_c = [&](int slot) __attribute__((always_inline)) {
        const T *c = ctile + (size_t)slot * WK * WV;
        if constexpr (C_REGS) {
#pragma unroll
            for (int ks = 0; ks < NKD; ++ks) cnext[ks] = gload<F>(c + 32 * w * WV + ks * E::KSTEP, (ln.r * WV + 8 * ln.h) * sizeof(T));
        } else {
            mc.template load_w<WV>(c, WK);   // rows and columns of padding read as zero
        }
    };
    auto store_c = [&]() __attribute__((always_inline)) {
        if constexpr (C_REGS) {
#pragma unroll
            for (int ks = 0; ks < NKD; ++ks) cf[ks] = cnext[ks];
        } else {
            mc.store(sC, LDD);
        }
    };
    // The requests for a pair come in two parts. K and V of both tiles go into registers that are idle
    // from the top of an iteration on, so inside the loop they are issued a whole tile early (during
    // the O tile of the pair before); dO, Q of the O tile and the cached state follow once the E tile
    // of the pair before has taken their registers' contents. Fewer requests are then issued in one
    // burst, which is where the waves stall at the memory pipeline's entry.
    auto load_pair_kv = [&](int tE) {
        mvO.template load_w<WV>(V + voff(tE + 1), nvalid(tE + 1));
        mkO.template load_w<WK>(K + koff(tE + 1), nvalid(tE + 1));
        mvE.template load_w<WV>(V + voff(tE), nvalid(tE));
        mkE.template load_w<WK>(K + koff(tE), nvalid(tE));
        if constexpr (!C_REGS) load_c(tE / 2);
    };
    auto load_pair_rest = [&](int tE) {
        const int nvO = nvalid(tE + 1);
        if constexpr (NORM) mnX.load(yn + voff(tE + 1), rstd_c + (size_t)(tE + 1) * CT, nvO);
        if constexpr (TOKEN) {
            // (a tile that is not there has no first token to read in place of the missing ones: log g = 0 throughout)
            if (!RAGGED || nvO > 0) lgO = TokenDecay<T, CT>::fetch(lg + (size_t)(tE + 1) * CT, nvO);
            else lgO = {};
            lgE = TokenDecay<T, CT>::fetch(lg + (size_t)tE * CT, nvalid(tE));
        }
        moX.template load_w<WV>(dO + voff(tE + 1), nvO);
        mqX.template load_w<WK>(Q + koff(tE + 1), nvO);
        if constexpr (C_REGS) load_c(tE / 2);
    };
    auto load_pair = [&](int tE) {
        load_pair_kv(tE);
        load_pair_rest(tE);
    };
    [[maybe_unused]] auto load_tile = [&](int t, int n) {   // by tiles
        mvE.template load_w<WV>(V + voff(t), n);
        mkE.template load_w<WK>(K + koff(t), n);
        moX.template load_w<WV>(dO + voff(t), n);
        mqX.template load_w<WK>(Q + koff(t), n);
        load_c(t);
        if constexpr (NORM) mnX.load(yn + voff(t), rstd_c + (size_t)t * CT, n);
        if constexpr (TOKEN) lgE = TokenDecay<T, CT>::fetch(lg + (size_t)t * CT, n);
    };
    [[maybe_unused]] auto load_half = [&](int t) __attribute__((always_inline)) {   // halves
        const int tE = t & ~1, n = nvalid(t);
        if (t & 1) {
            mvO.template load_w<WV>(V + voff(t), n);
            mkO.template load_w<WK>(K + koff(t), n);
            if constexpr (TOKEN) lgO = TokenDecay<T, CT>::fetch(lg + (size_t)t * CT, n);
        }
        mvE.template load_w<WV>(V + voff(tE), nvalid(tE));
        mkE.template load_w<WK>(K + koff(tE), nvalid(tE));
        load_c(tE / 2);
        if constexpr (NORM) mnX.load(yn + voff(t), rstd_c + (size_t)t * CT, n);
        if constexpr (TOKEN) lgE = TokenDecay<T, CT>::fetch(lg + (size_t)tE * CT, nvalid(tE));
        moX.template load_w<WV>(dO + voff(t), n);
        mqX.template load_w<WK>(Q + koff(t), n);
    };
    auto load_first = [&]() __attribute__((always_inline)) {
        if constexpr (BY_TILES) load_tile(t1 - 1, nvalid(t1 - 1));
        else if constexpr (HALVES) load_half(t0);
        else load_pair(t1 - 2);
    };
    // what the state alone needs, of the tiles behind this segment that the workgroup takes it through
    auto load_qdo = [&](int t) __attribute__((always_inline)) {
        moX.template load_w<WV>(dO + voff(t), nvalid(t));
        mqX.template load_w<WK>(Q + koff(t), nvalid(t));
        if constexpr (NORM) mnX.load(yn + voff(t), rstd_c + (size_t)t * CT, nvalid(t));
        if constexpr (TOKEN) lgE = TokenDecay<T, CT>::fetch(lg + (size_t)t * CT, nvalid(t));
    };
    const int own = OWN && carry == kOwn ? ntiles - t1 : 0;   // tiles behind this segment that the workgroup takes the state through
    if (OWN && own) load_qdo(ntiles - 1);
    else load_first();

    const T *sX2 = rg ? sQ : sdO;    // intra operand and state-update B operand: [token][feature in w]
    const T *sUA = rg ? sdO : sQ;    // state-update A operand: [token][feature of the state rows]
    T *sPm = rg ? sDS : sS;          // masked score tile of this group's product
    T *gOut = rg ? dK : dV;

    // st[blk][i]: group 0: dKV[32 blk + acc_row(i)][32 w + r]; group 1: dKV[32 w + r][32 blk + acc_row(i)]
    f32x16 st[DB];
    {
        const float *states = scratch + (size_t)chain * nslots * WK * WV;
        auto load = [&](f32x16(&s)[DB], const float *g) {
            if (rg == 0) state_load_w<D, WK, WV>(ln, s, g, w);
            else state_load_t_w<D, WK, WV>(ln, s, g, w);
        };
        if (carry) {
            const Pieces pc(true, !OWN && carry == kCarriedPieces, shards, nseg, tiles_per_seg, ntiles);
            start_state<true, SHARED>(st, scratch + ((ptrdiff_t)chain * pc.slots - pc.base) * WK * WV, dkv_out ? dkv_out + (size_t)chain * WK * WV : nullptr,
                              SegDecay<TOKEN>(decay, seglog + ((ptrdiff_t)chain * pc.slots - pc.base), chain, H, pc.per_shard, pc.tiles * CT, ntok),
                              OWN && carry == kOwn ? pc.per_shard * shards - 1 : piece_of<true>(pc, shard, seg), pc.per_shard, pc.per_shard * shards, WK * WV, load);
        } else load(st, states + (size_t)slot0 * WK * WV);
        if (dkv_copy && slot0 == nslots - 1 && rg == 0) state_store_w<D, WK, WV>(ln, st, dkv_copy + (size_t)chain * WK * WV, w);
    }

    // masked score tiles of the tile whose V, K are at pV, pK (dO, Q in sdO, sQ): one 32x32 block per wave
    // The O tile's queries against the E tile's keys: dSX^T[j][i] = sum_c V_E[j][c] dO_O[i][c], all four
    // 32x32 blocks, weighted and stored as sDX[i][j]. Two blocks go to the two waves that have no
    // triangular block, one each to two waves of group 0.
    auto cross_scores = [&]() {
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
            const int owner = blk < 2 ? 6 + blk : blk;   // waves 6, 7, 2, 3
            if (owner % (2 * NW) != w8) continue;
            const int ib = blk >> 1, jb = blk & 1;
            f32x16 acc = {0}, acc2 = {0};
            pipelined<WV / E::KSTEP / 2>(   // (contraction over the real value features)
                [&](int s2) {
                    FragPair<FragPair<F>> f;
                    f.a.a = E::ld_kc(ln, sVE, LDD, 32 * jb, 2 * s2 * E::KSTEP);
                    f.a.b = E::ld_kc(ln, sdO, LDD, 32 * ib, 2 * s2 * E::KSTEP);
                    f.b.a = E::ld_kc(ln, sVE, LDD, 32 * jb, (2 * s2 + 1) * E::KSTEP);
                    f.b.b = E::ld_kc(ln, sdO, LDD, 32 * ib, (2 * s2 + 1) * E::KSTEP);
                    return f;
                },
                [&](int, const FragPair<FragPair<F>> &f) {
                    acc = E::mfma(f.a.a, f.a.b, acc);
                    acc2 = E::mfma(f.b.a, f.b.b, acc2);
                });
            acc += acc2;
            const int iq = 32 * ib + ln.r;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int j0 = 32 * jb + 8 * g + 4 * ln.h;
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = acc[4 * g + e] * cross_weight(iq, j0 + e);
                E::st4(SM::block(sDX, ib, jb) + lds_off(LDP, ln.r, j0 - 32 * jb), x[0], x[1], x[2], x[3]);
            }
        }
    };
    auto scores = [&](const auto &dec, const T *pV, const T *pK) {
        constexpr int NTRI = 3;
#pragma unroll
        for (int idx = 0; idx < 2 * NTRI; ++idx) {
            if (idx % (2 * NW) != w8) continue;
            const int tri = idx % NTRI, ib = tri == 0 ? 0 : 1, jb = tri == 2 ? 1 : 0;
            const T *sA = idx < NTRI ? pV : pK, *sB = idx < NTRI ? sdO : sQ;
            f32x16 acc = {0}, acc2 = {0};
            auto contract = [&](auto steps) __attribute__((always_inline)) {
                pipelined<decltype(steps)::value>(
                    [&](int s2) {
                        FragPair<FragPair<F>> f;
                        f.a.a = E::ld_kc(ln, sA, LDD, 32 * jb, 2 * s2 * E::KSTEP);
                        f.a.b = E::ld_kc(ln, sB, LDD, 32 * ib, 2 * s2 * E::KSTEP);
                        f.b.a = E::ld_kc(ln, sA, LDD, 32 * jb, (2 * s2 + 1) * E::KSTEP);
                        f.b.b = E::ld_kc(ln, sB, LDD, 32 * ib, (2 * s2 + 1) * E::KSTEP);
                        return f;
                    },
                    [&](int, const FragPair<FragPair<F>> &f) {
                        acc = E::mfma(f.a.a, f.a.b, acc);
                        acc2 = E::mfma(f.b.a, f.b.b, acc2);
                    });
            };
            // dS = dO V^T contracts over the real value features, S = Q K^T over the real key features
            if (idx < NTRI) contract(std::integral_constant<int, WV / E::KSTEP / 2>{});
            else contract(std::integral_constant<int, WK / E::KSTEP / 2>{});
            acc += acc2;
            store_masked_scores<T, LDP>(ln, SM::block(idx < NTRI ? sDS : sS, ib, jb), acc, jb, ib, dec);
        }
    };

    // dQ, this group's dV or dK, and the dKV update for tile `t`
    // `cross` (the O tile): the cached state is the one the E tile starts from, so dQ takes the E tile
    // as the first half of its own chunk: far weights on the state term, plus the E tile's keys through sDX.
    // Key and value dimensions that differ: only KB (VB) of the DB 32-wide feature blocks of the key (value)
    // side are real. A wave whose own output block (dV block w in group 0, dK block w in group 1) is padding
    // skips that product and its state update. With d_k < d_v the two such waves of group 1 produce ALL of
    // dQ instead (both token blocks of one key-feature block each), so that no wave carries dQ on top of a
    // dK or dV block and a state update (the walk's critical path); otherwise every wave with a real
    // key-feature block produces the dQ tile of that block for one token block (group 0 the second, whose
    // keys span both blocks, group 1 the first).
    constexpr int KB = WK / 32, VB = WV / 32;
    const bool own_block = WK == WV || (rg ? w < KB : w < VB);   // this wave's dK / dV block exists
    auto update = [&](const auto &dec, int nrows) __attribute__((always_inline)) {
        if (own_block) {   // state update in this group's orientation
            const float lamC = dec.whole(nrows);
#pragma unroll
            for (int blk = 0; blk < DB; ++blk) st[blk] *= lamC;
            struct Step { F b; F a[DB]; };
            pipelined<NKS>(
                [&](int ks) {
                    Step f;
                    f.b = E::ld_ks(ln, sX2, LDD, ks * E::KSTEP, 32 * w);
#pragma unroll
                    for (int blk = 0; blk < DB; ++blk) f.a[blk] = E::ld_ks(ln, sUA, LDD, ks * E::KSTEP, 32 * blk);
                    return f;
                },
                [&](int ks, const Step &f) {
                    const F bs = dec.weigh_upto(ln, f.b, ks);
#pragma unroll
                    for (int blk = 0; blk < DB; ++blk) st[blk] = E::mfma(f.a[blk], bs, st[blk]);
                });
        }
    };
    if constexpr (OWN)
    for (int t = ntiles - 1; t >= ntiles - own; --t) {
        __syncthreads();
        if constexpr (NORM) mnX.apply(moX);
        moX.store(sdO, LDD);
        mqX.store(sQ, LDD);
        if constexpr (TOKEN) decE.fill(lgE);
        __syncthreads();
        if (t > t1) load_qdo(t - 1);
        else load_first();
        ln = fresh_lane();
        update(decE, nvalid(t));
    }
    constexpr bool DQ_BY_IDLE = WK < WV && !(TOKEN && NORM);   // (that one combination would run out of registers)
    auto products = [&](const auto &dec, const T *pV, const T *pK, int t, int nrows, bool cross) {
        const T *sX1 = rg ? pV : pK;  // inter operand: token rows, features contracted with the state
        float rq[NB] = {};  // per-token decay: q_i . dq_i over the features of the dQ tiles this wave produced, per token block
        // dQ^T[a in block qa][i], tokens i of the block starting at r0; `both`: the intra part reaches the keys of
        // both blocks (the second token block) or of block 0 only
        auto dq_tile = [&](int qa, int r0, auto both) __attribute__((always_inline)) {
            f32x16 acc = {0};
            pipelined<WV / E::KSTEP>(   // (the cached state's real columns)
                [&](int ks) {
                    FragPair<F> f;
                    if constexpr (C_REGS) f.a = cf[ks];   // (qa = w)
                    else f.a = E::ld_kc(ln, sC, LDD, 32 * qa, ks * E::KSTEP);
                    f.b = E::ld_kc(ln, sdO, LDD, r0, ks * E::KSTEP);
                    return f;
                },
                [&](int, const FragPair<F> &f) { acc = E::mfma(f.a, f.b, acc); });
            acc *= cross ? far_upto(r0 + ln.r) : dec.upto(r0 + ln.r);
            auto fma = [&](int, const FragPair<F> &f) { acc = E::mfma(f.a, f.b, acc); };
            if (cross)
                pipelined<NKS>(
                    [&](int ks) { return FragPair<F>{E::ld_ks(ln, sKE, LDD, ks * E::KSTEP, 32 * qa), E::ld_kc(ln, SM::block(sDX, r0 / 32, ks / SPB), LDP, 0, ks % SPB * E::KSTEP)}; },
                    fma);
            auto intra = [&](int ks) { return FragPair<F>{E::ld_ks(ln, pK, LDD, ks * E::KSTEP, 32 * qa), E::ld_kc(ln, SM::block(sDS, r0 / 32, ks / SPB), LDP, 0, ks % SPB * E::KSTEP)}; };
            pipelined<decltype(both)::value ? 2 * SPB : SPB>(intra, fma);
            if constexpr (TOKEN) rq[r0 / 32] = rowdot<T>(ln, acc, sQ, LDD, r0, qa);   // (from the fp32 accumulators, before rounding)
            store_out_tile_t<T, D, WK>(ln, dQ + koff(t), acc, r0, qa, nrows);
        };
        if constexpr (DQ_BY_IDLE) {
            if (rg == 1 && w >= KB) {
                dq_tile(w - KB, 32, std::true_type{});
                dq_tile(w - KB, 0, std::false_type{});
            }
        } else if (WK == WV || w < KB) {
            if (rg == 0) dq_tile(w, 32, std::true_type{});
            else dq_tile(w, 0, std::false_type{});
        }
        ln = fresh_lane();
        if (own_block) {   // dV^T[c in w][j] (group 0) or dK^T[a in w][j] (group 1), both token blocks
            f32x16 acc[NB];
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) acc[jb] = f32x16{0};
            struct Two { F b[NB]; };
            pipelined<DB * E::NSUB>(
                [&](int s2) {
                    Two f;
#pragma unroll
                    for (int jb = 0; jb < NB; ++jb) f.b[jb] = E::ld_kp(ln, sX1, LDD, 32 * jb, 32 * (s2 / E::NSUB), s2 % E::NSUB);
                    return f;
                },
                [&](int s2, const Two &f) {
                    const F sf = E::from_acc(st[s2 / E::NSUB], s2 % E::NSUB);
#pragma unroll
                    for (int jb = 0; jb < NB; ++jb) acc[jb] = E::mfma(sf, f.b[jb], acc[jb]);
                });
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) acc[jb] *= dec.after(32 * jb + ln.r, nrows);
            struct Three { F a; F b[NB]; };
            pipelined<NKS>(
                [&](int ks) {
                    Three f;
                    f.a = E::ld_ks(ln, sX2, LDD, ks * E::KSTEP, 32 * w);
#pragma unroll
                    for (int jb = 0; jb < NB; ++jb)
                        if (jb <= ks / SPB) f.b[jb] = E::ld_ks(ln, SM::block(sPm, ks / SPB, jb), LDP, ks % SPB * E::KSTEP, 0);
                    return f;
                },
                [&](int ks, const Three &f) {
#pragma unroll
                    for (int jb = 0; jb < NB; ++jb)
                        if (jb <= ks / SPB) acc[jb] = E::mfma(f.a, f.b[jb], acc[jb]);
                });
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
                if constexpr (TOKEN) {   // (row dots from the fp32 accumulators, before they are rounded and stored)
                    float r = rq[jb];
                    if (rg == 1) r -= rowdot<T>(ln, acc[jb], pK, LDD, 32 * jb, w);  // group 1 holds dK
                    if (ln.h == 0) rs[w8 * CT + 32 * jb + ln.r] = r;
                }
                if constexpr (WK == WV) {
                    store_out_tile_t<T, D, WK>(ln, gOut + koff(t), acc[jb], 32 * jb, w, nrows);
                } else {
                    if (rg) store_out_tile_t<T, D, WK>(ln, dK + koff(t), acc[jb], 32 * jb, w, nrows);
                    else store_out_tile_t<T, D, WV>(ln, dV + voff(t), acc[jb], 32 * jb, w, nrows);
                }
            }
        } else if constexpr (TOKEN) {   // this wave's row of the per-token sums still has to be defined
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
                if (ln.h == 0) rs[w8 * CT + 32 * jb + ln.r] = rq[jb];
        }
        ln = fresh_lane();
        update(dec, nrows);
    };

    if constexpr (BY_TILES) {
        for (int t = t1 - 1; t >= t0; --t) {
            __syncthreads();  // previous tile fully consumed
            ln = fresh_lane();
            if constexpr (TOKEN) {
                if (t + 1 < t1) flush_r(t + 1);
                decE.fill(lgE);
            }
            if constexpr (NORM) mnX.apply(moX);
            mvE.store(sVE, LDD);
            moX.store(sdO, LDD);
            mkE.store(sKE, LDD);
            mqX.store(sQ, LDD);
            store_c();
            __syncthreads();
            ln = fresh_lane();
            if (t > t0) load_tile(t - 1, CT);   // (only the sub-sequence's last tile is short)
            scores(decE, sVE, sKE);
            __syncthreads();
            ln = fresh_lane();
            products(decE, sVE, sKE, t, nvalid(t), false);
        }
    }
    if constexpr (HALVES) {
        const bool odd = t0 & 1;
        const auto dec = [&] {
            if constexpr (TOKEN) return TokenDecay<T, CT>(odd ? pw : pw + 3 * CT);
            else return decO;
        }();
        const T *pV = odd ? sVO : sVE, *pK = odd ? sKO : sKE;
        __syncthreads();
        ln = fresh_lane();
        if constexpr (TOKEN) {
            if (odd) decO.fill(lgO);
            decE.fill(lgE);
        }
        if constexpr (NORM) mnX.apply(moX);
        if (odd) {
            mvO.store(sVO, LDD);
            mkO.store(sKO, LDD);
        }
        moX.store(sdO, LDD);
        mqX.store(sQ, LDD);
        mvE.store(sVE, LDD);
        mkE.store(sKE, LDD);
        store_c();
        __syncthreads();
        ln = fresh_lane();
        scores(dec, pV, pK);
        if (odd) cross_scores();
        __syncthreads();
        ln = fresh_lane();
        products(dec, pV, pK, t0, nvalid(t0), odd);
    }
    for (int tE = MODE != kPairs ? t0 - 1 : t1 - 2; tE >= t0; tE -= 2) {
        __syncthreads();  // previous pair fully consumed
        ln = fresh_lane();
        if constexpr (TOKEN) {
            if (tE + 2 < t1) flush_r(tE + 2);  // E tile of the previous pair
            decO.fill(lgO);
            decE.fill(lgE);
        }
        if constexpr (NORM) mnX.apply(moX);
        mvO.store(sVO, LDD);
        moX.store(sdO, LDD);
        mkO.store(sKO, LDD);
        mqX.store(sQ, LDD);
        mvE.store(sVE, LDD);
        mkE.store(sKE, LDD);
        store_c();   // the state the E tile starts from serves both tiles of the pair
        if (tE > t0) load_pair_kv(tE - 2);
        __syncthreads();
        ln = fresh_lane();
        moX.template load_w<WV>(dO + voff(tE), nvalid(tE));
        mqX.template load_w<WK>(Q + koff(tE), nvalid(tE));
        if constexpr (NORM) mnX.load(yn + voff(tE), rstd_c + (size_t)tE * CT, nvalid(tE));
        // ---- O tile ----
        const int nvO = nvalid(tE + 1);
        if (!RAGGED || nvO > 0) {
            scores(decO, sVO, sKO);
            cross_scores();
            __syncthreads();
            ln = fresh_lane();
            products(decO, sVO, sKO, tE + 1, nvO, true);
            __syncthreads();  // O tile consumed: sdO, sQ are free
            ln = fresh_lane();
            if constexpr (TOKEN) flush_r(tE + 1);
        }
        if constexpr (NORM) mnX.apply(moX);
        moX.store(sdO, LDD);
        mqX.store(sQ, LDD);
        __syncthreads();
        ln = fresh_lane();
        if (tE > t0) load_pair_rest(tE - 2);
        // ---- E tile ----
        scores(decE, sVE, sKE);
        __syncthreads();
        ln = fresh_lane();
        products(decE, sVE, sKE, tE, nvalid(tE), false);
    }
    if constexpr (TOKEN) {
        __syncthreads();
        flush_r(t0);
    }
    if (seg == 0 && rg == 0) state_store_w<D, WK, WV>(ln, st, dkv_in + (size_t)chain * WK * WV, w);
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
template <typename T, int CT, int D>
struct Smem {
    static constexpr size_t tile = (size_t)walk_tile<T>(CT, walk_ld<T, D>()) * sizeof(bf16_t),
                            scores = (size_t)(walk_tile<T>(CT, fwd_ldp<T, CT>()) + fwd_stage<T, D>()) * sizeof(bf16_t),
                            tables = table_floats<CT>() * sizeof(float);
    static constexpr size_t local = 2 * tile + tables;
    static constexpr size_t fwd = 3 * tile + scores + tables;
};

// One launch of a kernel with `lds` bytes of dynamic LDS. Kernels that need more than the 64 KB default
// have their limit raised first (once per kernel and device, see allow_dynamic_lds).
template <typename... KArgs, typename... Args>
static hipError_t launch_kernel(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t s, Args... args) {
    if (hipError_t e = allow_dynamic_lds((const void *)kernel, lds); e != hipSuccess) return e;
    kernel<<<grid, block, lds, s>>>(args...);
    return hipSuccess;
}

// A kernel family instantiated for both decay models, with and without a short last tile (or an odd tile
// count, where tiles are walked in pairs), with and without the fused Norm: picks the member that serves the
// plan. Fam::fn<TOKEN, RAGGED, NORM> is the kernel. The kernels for whole tiles know every row count at
// compile time: with the row checks in them the walks lose 1 %, and 3-4 % where they are short (c2's shards
// 154 -> 161 us a step).
template <typename Fam, bool TK>
static auto by_edges(const Plan &p) {
    return p.ragged ? (p.norm ? Fam::template fn<TK, true, true> : Fam::template fn<TK, true, false>)
                    : (p.norm ? Fam::template fn<TK, false, true> : Fam::template fn<TK, false, false>);
}
// (launches that several sub-sequences share know one lambda per head only)
template <typename Fam>
static auto by_model(const Plan &p) {
    if constexpr (Fam::kShared) return by_edges<Fam, false>(p);
    else return p.token ? by_edges<Fam, true>(p) : by_edges<Fam, false>(p);
}
// go(sh) with the distances of a launch's sub-sequences, or with Alone for a launch of one: those are kernels of their own,
// whose arguments do not hold the distances (128 - 350 bytes a launch, 0.1 - 0.2 us: three launches of a float forward pass
// over 2 heads x 256 tokens, d=64, through the Python binding 14.59 us with the distances, 13.97 without).
template <typename SH, typename Go>
static hipError_t by_shards(const Plan &p, const SH &sh, Go go) { return p.shards > 1 ? go(sh) : go(Alone{}); }
// The walks also with AloneOwn, where the workgroups compute their start states: with the loop that does it in every walk the
// forward one at d=64 takes longer, 16 heads x 710 tokens 8.8 -> 9.3 us, 32 x 8448 with a decay per token 48.0 -> 49.1.
template <typename SH, typename Go>
static hipError_t by_start(const Plan &p, Start start, const SH &sh, Go go) { return start == kOwn ? go(AloneOwn{}) : by_shards(p, sh, go); }

// Kernel families by decay model and Norm (see by_model).
template <typename SH>
struct Family {
    static constexpr bool kShared = is_shared<SH>;
};
template <typename T, int CT, int D, bool BWD, int WX, int WY, typename SH, int G>
struct LocalFam : Family<SH> {   // the Norm prologue exists in the backward pass only; alone the forward pass never sums over a short end
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_local<T, CT, D, BWD, TK, RG && (BWD || is_shared<SH>), NM && BWD, WX, WY, SH, G>;
};
template <typename T, int CT, int D, int WK, int WV, typename SH>
struct FwdFam : Family<SH> {
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_fwd<T, CT, D, TK, RG, NM, WK, WV, kOutputs, SH>;
};
template <typename T, int CT, int D, int WK, int WV, typename SH>
struct StatesFam : Family<SH> {  // the forward walk reduced to the states (no Norm: the states do not depend on it)
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_fwd<T, CT, D, TK, RG, false, WK, WV, kStates, SH>;
};
template <typename T, int CT, int D, Role ROLE, typename SH>
struct Fwd8Fam : Family<SH> {
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_fwd8<T, CT, D, TK, RG, NM && ROLE == kOutputs, ROLE, SH>;
};
template <typename T, int CT, int D, int WK, int WV, typename SH>
struct DqFam : Family<SH> {      // dQ as a forward walk over dO, V, K
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_fwd<T, CT, D, TK, RG, NM, WV, WK, kDq, SH>;
};
template <typename T, int CT, int D, int WK, int WV, typename SH>
struct BwdkvFam : Family<SH> {
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_bwdkv<T, CT, D, TK, RG, NM, WK, WV, SH>;
};
template <typename T, int CT, int D, int WK, int WV, typename SH>
struct Bwd8pFam : Family<SH> {   // eight waves, one cached state per pair of tiles
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_bwd8p<T, CT, D, TK, RG, NM, WK, WV, kPairs, SH>;
};
template <typename T, int CT, int D, int WK, int WV, typename SH>
struct Bwd8tFam : Family<SH> {   // one cached state per tile; an odd tile count is ragged
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_bwd8p<T, CT, D, TK, true, NM, WK, WV, kTiles, SH>;
};
template <typename T, int CT, int D, int WK, int WV>
struct Bwd8hFam : Family<AloneOwn> {   // one cached state per pair of tiles, a workgroup per tile
    template <bool TK, bool RG, bool NM>
    static constexpr auto fn = k_bwd8p<T, CT, D, TK, true, NM, WK, WV, kHalves, AloneOwn>;
};

// The local pass only sums over its segment, so its tile need not be the walk's:
// bfloat16 segments of an even number of 64-token tiles are read 128 tokens
// at a time (half the barriers, twice the bytes in flight per workgroup), unless
// key and value dimensions that differ ask for the walk's tile. Two groups of waves where the dimensions are the same, half of
// the state's rows each: a second wave per SIMD to run while one waits, half of the stores into LDS (and of Norm's
// arithmetic) a wave. Steps, d=128, one group / two: 16 heads x 8192 tokens 156.5 / 151.4 us, 32 x 2048 98.8 / 95.3, 2 x 16 x 5000 with
// states 181.0 / 175.6, Norm 16 x 8192 (64-token tiles / 128) 170.2 / 164.6; d=64 16 x 8192
// 79.9 / 78.1, 32 x 2048 57.5 / 56.3; of 48 to 256 heads x 256 to 2048 tokens, with Norm and a decay per token too, none is slower.
// The forward pass of one sub-sequence never sums over the segment with the short end.
template <typename T, int CT, int D, bool BWD, int WK = D, int WV = D>
static hipError_t run_local(const Plan &p, const T *x, const T *y, const float *decay, float *scratch, float *seglog,
                            const T *yn, const float *rstd, Start start, const Shards &all, hipStream_t s) {
    constexpr int G = sizeof(T) == 2 && WK == D && WV == D ? 2 : 1;
    const LocalShards sh{BWD ? all.q : all.k, BWD ? all.dout : all.v, all.yn, all.rstd};
    const Pieces pc(BWD, start == kCarriedPieces, p.shards, p.nseg, p.tiles_per_seg, p.ntiles);
    const int segs = pc.n == 2 ? -p.nseg : p.nseg;
    const dim3 grid(p.shards > 1 ? pc.per_shard : pc.end - pc.first, p.B * p.H, p.shards), block(D * 2 * G);
    Plan q = p;
    if constexpr (G == 2 && CT == 64) {
        if (pc.tiles % 2 == 0) {
            if (!BWD) q.ragged = p.N % 128 != 0;
            return by_shards(p, sh, [&](auto of) {
                return launch_kernel(by_model<LocalFam<T, 128, D, BWD, D, D, decltype(of), G>>(q), grid, block, Smem<T, 128, D>::local, s, x, y,
                                     decay, scratch, seglog, p.H, (p.ntiles + 1) / 2, segs, p.tiles_per_seg / 2, p.N, p.kvdiv, yn, rstd, of);
            });
        }
    }
    return by_shards(p, sh, [&](auto of) {
        return launch_kernel(by_model<LocalFam<T, CT, D, BWD, WK, WV, decltype(of), G>>(q), grid, block, Smem<T, CT, D>::local, s, x, y, decay,
                             scratch, seglog, p.H, p.ntiles, segs, p.tiles_per_seg, p.N, p.kvdiv, yn, rstd, of);
    });
}

// Where the walk's start states come from: own_states (lasp_rules.h) where the plan says so; else, up to four segments, the
// walk carries the boundary state over the local states before its own (start_state) instead of a scan kernel filling
// every segment's slot. Each segment carried over costs the walk 1.3 - 1.8 us before its
// first tile (a state's loads, one after the other), the scan 3 - 11 us and a launch. bf16 d=128 forward / backward:
// 128 heads x 1024 tokens (2 segments) 63.9 / 88.2 -> 56.8 / 79.2 us, 64 x 8192 (4) 195.4 / 302.4 -> 188.0 / 301.9,
// but 16 x 1024 (8) 31.7 / 37.3 -> 39.7 / 47.3.
static Start walk_start(const Plan &p) {
    if (p.own_states) return kOwn;
    if (p.shards * p.nseg > 4) return kScanned;
    return local_pieces(p.shards * p.nseg, p.tiles_per_seg, (long long)p.B * p.H) == 2 ? kCarriedPieces : kCarried;
}

// Local pass and scan of the forward states over K, V, as far as the walk's start asks for them.
template <typename T, int CT, int D, int WK, int WV>
static hipError_t run_states(const Plan &p, const void *k, const void *v, const float *kv_in, const float *decay, float *scratch,
                             float *seglog, Start start, const Shards &sh, hipStream_t s, const KernelEvents *ke) {
    if (start != kOwn && p.shards * p.nseg > 1) {
        if (hipError_t e = run_local<T, CT, D, false, WK, WV>(p, (const T *)k, (const T *)v, decay, scratch, seglog, nullptr, nullptr, start, sh, s);
            e != hipSuccess)
            return e;
    }
    if (ke) (void)hipEventRecord(ke->ev[1], s);
    return start != kScanned ? hipSuccess : launch_scan(p, false, scratch, kv_in, decay, seglog, s);
}

template <typename T, int CT, int D, int WK = D, int WV = D>
static hipError_t run_fwd(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) {
    const Start start = walk_start(p);
    hipError_t e;
    if (ke) (void)hipEventRecord(ke->ev[0], s);
    if (e = run_states<T, CT, D, WK, WV>(p, a.k, a.v, a.kv_in, a.decay, a.scratch, a.seglog, start, a.sh, s, ke); e != hipSuccess) return e;
    if (ke) (void)hipEventRecord(ke->ev[2], s);
    static_assert(Smem<T, CT, D>::fwd <= 163840 / 2, "two workgroups of the walk share a CU's LDS");
    const FwdShards sh{a.sh.q, a.sh.k, a.sh.v, a.sh.cache, a.sh.out, a.sh.rstd, a.sh.kv_out, {}};
    const dim3 grid(p.nseg, p.B * p.H, p.shards);
    if constexpr (sizeof(T) == 2 && WK == 128 && WV == 128) {
        static_assert(Fwd8Smem<T, CT, D>::TOTAL <= 163840, "LDS budget of one gfx950 CU exceeded");
        // Up to 256 workgroups a CU has one, and four waves leave each SIMD only one; from 257 on two workgroups of
        // k_fwd share a CU (70 KB of LDS each; k_fwd8 takes 112), need no exchange and do not wait for each other.
        // Forward, k_fwd / k_fwd8, us: 256 workgroups, 128 heads x 8192 tokens 309.0 / 300.1, x 4000 165.0 / 156.4,
        // x 8192 with a decay per token 357.6 / 315.2; 512 workgroups, 512 heads x 2048 221.7 / 235.7, x 2000
        // 231.3 / 238.8, x 2048 with a decay per token 223.0 / 253.3.
        if ((int64_t)p.shards * p.nseg * p.B * p.H <= kOnePerCu) {
            e = by_start(p, start, sh, [&](auto of) {
                using SH = decltype(of);
                const auto walk8 = a.states_only ? by_model<Fwd8Fam<T, CT, D, kStates, SH>>(p) : by_model<Fwd8Fam<T, CT, D, kOutputs, SH>>(p);
                return launch_kernel(walk8, grid, dim3(D * 4), Fwd8Smem<T, CT, D>::TOTAL, s, (const T *)a.q,
                                     (const T *)a.k, (const T *)a.v, a.decay, (T *)a.out, a.kv_out, (T *)a.cache, p.cache_tiles,
                                     (const float *)a.scratch, a.kv_in, (const float *)a.seglog, (int)start, p.H, p.ntiles, p.nseg,
                                     p.tiles_per_seg, p.N, p.kvdiv, a.rstd_out, a.eps, a.kv_copy, of);
            });
            if (e != hipSuccess) return e;
            if (ke) (void)hipEventRecord(ke->ev[3], s);
            return hipGetLastError();
        }
    }
    e = by_start(p, start, sh, [&](auto of) {
        using SH = decltype(of);
        const auto walk = a.states_only ? by_model<StatesFam<T, CT, D, WK, WV, SH>>(p) : by_model<FwdFam<T, CT, D, WK, WV, SH>>(p);
        return launch_kernel(walk, grid, dim3(D * 2), Smem<T, CT, D>::fwd, s,
                             (const T *)a.q, (const T *)a.k, (const T *)a.v, a.decay, (T *)a.out, a.kv_out, (T *)a.cache,
                             p.cache_tiles, (const float *)a.scratch, a.kv_in, (const float *)a.seglog, (int)start, p.H, p.ntiles, p.nseg,
                             p.tiles_per_seg, p.N, p.kvdiv, a.rstd_out, a.eps, (const T *)nullptr, (const float *)nullptr,
                             (const T *)nullptr, (float *)nullptr, a.kv_copy, of);
    });
    if (e != hipSuccess) return e;
    if (ke) (void)hipEventRecord(ke->ev[3], s);
    return hipGetLastError();
}

// dQ of float data: from the states the forward pass kept (a.cache), or, when it is given none, from the
// states rebuilt into the scratch buffer, which the backward states overwrite afterwards.
template <typename T, int CT, int D, int WK, int WV>
static hipError_t run_dq(const BwdArgs &a, hipStream_t s) {
    const Plan &f = *a.fwd;   // a segment per cached state
    const Start start = a.cache ? kKept : walk_start(f);   // kKept: a state per segment of every sub-sequence, in its own buffer
    if (!a.cache) {
        if (hipError_t e = run_states<T, CT, D, WK, WV>(f, a.k, a.v, a.kv_in, a.decay, a.scratch, a.seglog, start, a.sh, s, nullptr);
            e != hipSuccess)
            return e;
    }
    return by_start(f, start, FwdShards{a.sh.dout, a.sh.v, a.sh.k, a.sh.cache, a.sh.dq, a.sh.rstd, {}, a.sh.yn}, [&](auto of) {
        return launch_kernel(by_model<DqFam<T, CT, D, WK, WV, decltype(of)>>(f), dim3(f.nseg, f.B * f.H, f.shards), dim3(D * 2), Smem<T, CT, D>::fwd,
                             s, (const T *)a.dout, (const T *)a.v, (const T *)a.k, a.decay, (T *)a.dq, (float *)nullptr, (T *)nullptr,
                             f.cache_tiles, a.cache ? (const float *)a.cache : (const float *)a.scratch, a.kv_in, (const float *)a.seglog,
                             (int)start, f.H, f.ntiles, f.nseg, f.tiles_per_seg, f.N, f.kvdiv, (float *)nullptr, 0.0f, (const T *)a.yn, a.rstd,
                             (const T *)a.q, a.rtok, (float *)nullptr, of);
    });
}

template <typename T, int CT, int D, int WK = D, int WV = D>
static hipError_t run_bwd(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) {
    const int chains = p.B * p.H;
    const Start start = walk_start(p);
    hipError_t e;
    if (ke) (void)hipEventRecord(ke->ev[0], s);
    if constexpr (sizeof(T) == 4) {
        if (!a.cache) {
            if (e = run_dq<T, CT, D, WK, WV>(a, s); e != hipSuccess) return e;
        }
    }
    if (start != kOwn && p.shards * p.nseg > 1) {
        if (e = run_local<T, CT, D, true, WK, WV>(p, (const T *)a.q, (const T *)a.dout, a.decay, a.scratch, a.seglog, (const T *)a.yn,
                                          a.rstd, start, a.sh, s);
            e != hipSuccess)
            return e;
    }
    if (ke) (void)hipEventRecord(ke->ev[1], s);
    if (start == kScanned) {
        if (e = launch_scan(p, true, a.scratch, a.dkv_out, a.decay, a.seglog, s); e != hipSuccess) return e;
    }
    if (ke) (void)hipEventRecord(ke->ev[2], s);
    // The walks: bfloat16 in one kernel with one cached state per pair of tiles; float dQ and dK, dV apart.
    const dim3 grid(p.nseg, chains, p.shards), block(D * 4);
    const BwdShards sh{a.sh.q, a.sh.k, a.sh.v, a.sh.dout, a.sh.cache, a.sh.dq, a.sh.dk, a.sh.dv, a.sh.dkv_in, a.sh.yn, a.sh.rstd};
    if constexpr (sizeof(T) == 2) {
        static_assert(Bwd8pSmem<T, CT, D>::TOTAL <= 163840, "LDS budget of one gfx950 CU exceeded");
        static_assert(D != 64 || (Bwd8pSmem<T, CT, D>::TOTAL <= 163840 / 2 && Bwd8pSmem<T, CT, D, kTiles>::TOTAL <= 163840 / 2),
                      "two workgroups share a CU at d=64");
        const bool by_tiles = p.cache_tiles == 1;
        auto go = [&](auto of) {
            using SH = decltype(of);
            const auto walk = by_tiles ? by_model<Bwd8tFam<T, CT, D, WK, WV, SH>>(p) : [&] {
                if constexpr (is_own<SH>) return by_model<Bwd8hFam<T, CT, D, WK, WV>>(p);
                else return by_model<Bwd8pFam<T, CT, D, WK, WV, SH>>(p);
            }();
            return launch_kernel(walk, grid, block, by_tiles ? Bwd8pSmem<T, CT, D, kTiles>::TOTAL : is_own<SH> ? Bwd8pSmem<T, CT, D, kHalves>::TOTAL : Bwd8pSmem<T, CT, D>::TOTAL, s, (const T *)a.q,
                                 (const T *)a.k, (const T *)a.v, (const T *)a.dout, a.decay, (const T *)a.cache, (T *)a.dq, (T *)a.dk,
                                 (T *)a.dv, a.dkv_in, (const float *)a.scratch, a.dkv_out, (const float *)a.seglog, (int)start, a.rtok, p.H,
                                 p.ntiles, p.nseg, p.tiles_per_seg, p.N, p.kvdiv, (const T *)a.yn, a.rstd, a.dkv_copy, of);
        };
        // (single tiles of pairs: also a sequence of one tile, whose workgroups have no tile behind them)
        e = !by_tiles && p.tiles_per_seg == 1 ? go(AloneOwn{}) : by_start(p, start, sh, go);
    } else {
        static_assert(BwdkvSmem<T, CT, D>::TOTAL <= 163840 / (D == 128 ? 1 : 2), "LDS of one gfx950 CU for the workgroups meant to share it");
        if (a.cache) {
            if (e = run_dq<T, CT, D, WK, WV>(a, s); e != hipSuccess) return e;
        }
        e = by_start(p, start, sh, [&](auto of) {
            return launch_kernel(by_model<BwdkvFam<T, CT, D, WK, WV, decltype(of)>>(p), grid, block, BwdkvSmem<T, CT, D>::TOTAL, s, (const T *)a.q,
                                 (const T *)a.k, (const T *)a.v, (const T *)a.dout, a.decay, (T *)a.dk, (T *)a.dv, a.dkv_in,
                                 (const float *)a.scratch, a.dkv_out, (const float *)a.seglog, (int)start, a.rtok, p.H, p.ntiles, p.nseg,
                                 p.tiles_per_seg, p.N, p.kvdiv, (const T *)a.yn, a.rstd, a.dkv_copy, of);
        });
    }
    if (e != hipSuccess) return e;
    if (p.kvdiv > 1) {
        if (e = launch_group_sum(p, a, s); e != hipSuccess) return e;
    }
    if (ke) (void)hipEventRecord(ke->ev[3], s);
    if (p.token) return launch_dlg(p, a, s);
    return hipGetLastError();
}

// One translation unit per combination of data type and dimensions (LASP_UNIT), so that they compile side by side.
#if LASP_UNIT == 0
hipError_t fwd_f32_64(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_fwd<float, 32, 64>(p, a, s, ke); }
hipError_t bwd_f32_64(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_bwd<float, 32, 64>(p, a, s, ke); }
#elif LASP_UNIT == 1
hipError_t fwd_f32_128(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_fwd<float, 32, 128>(p, a, s, ke); }
hipError_t bwd_f32_128(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_bwd<float, 32, 128>(p, a, s, ke); }
#elif LASP_UNIT == 2
hipError_t fwd_f32_64_128(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_fwd<float, 32, 128, 64, 128>(p, a, s, ke); }
hipError_t bwd_f32_64_128(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_bwd<float, 32, 128, 64, 128>(p, a, s, ke); }
#elif LASP_UNIT == 3
hipError_t fwd_f32_128_64(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_fwd<float, 32, 128, 128, 64>(p, a, s, ke); }
hipError_t bwd_f32_128_64(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_bwd<float, 32, 128, 128, 64>(p, a, s, ke); }
#elif LASP_UNIT == 4
hipError_t fwd_bf16_64(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_fwd<bf16_t, 64, 64>(p, a, s, ke); }
hipError_t bwd_bf16_64(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_bwd<bf16_t, 64, 64>(p, a, s, ke); }
#elif LASP_UNIT == 5
hipError_t fwd_bf16_128(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_fwd<bf16_t, 64, 128>(p, a, s, ke); }
hipError_t bwd_bf16_128(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_bwd<bf16_t, 64, 128>(p, a, s, ke); }
#elif LASP_UNIT == 6
hipError_t fwd_bf16_64_128(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_fwd<bf16_t, 64, 128, 64, 128>(p, a, s, ke); }
hipError_t bwd_bf16_64_128(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_bwd<bf16_t, 64, 128, 64, 128>(p, a, s, ke); }
#elif LASP_UNIT == 7
hipError_t fwd_bf16_128_64(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_fwd<bf16_t, 64, 128, 128, 64>(p, a, s, ke); }
hipError_t bwd_bf16_128_64(const Plan &p, const BwdArgs &a, hipStream_t s, const KernelEvents *ke) { return run_bwd<bf16_t, 64, 128, 128, 64>(p, a, s, ke); }
#else
#error "LASP_UNIT selects the instances of this translation unit: 0 .. 7"
#endif

}  // namespace lasp
