// HIP kernels (gfx950 / CDNA4) for bidirectional (unmasked) linear attention,
// the right-product form O = Q (K^T V) of LASP (arxiv 2404.02882) Sec. 3.1,
// Eq. (3), without the Norm. There is no mask, no decay and no order among the
// tokens, so the path is two streaming passes:
//   k_bidir_reduce + k_bidir_sum : the d x d state, a plain sum over tokens,
//       state = sum_s x_s y_s^T (K^T V forward, Q^T dO backward). Every head is
//       cut into segments whose partial sums are added in a fixed order (no
//       atomics: results are bit-reproducible).
//   k_bidir_apply : Out = X S or X S^T for a d x d state held in registers,
//       forward O = Q KV; backward dQ = dO KV^T, dK = V dKV^T, dV = K dKV (the
//       three as one launch). Where a whole sequence is at hand (lasp_bidir_seq_bwd)
//       dQ, which does not wait for dKV, comes from the reduction instead, which has
//       dO on chip, and up to four sub-sequences share every launch.
// Wave tiling and MFMA shapes as in lasp_walks.hip: wave w owns the 32-wide
// column block w of the state and of every output tile.
#include <hip/hip_runtime.h>

#include "lasp_internal.h"
#include "lasp_rules.h"
#include "lasp_device.h"

namespace lasp {

// Sub-sequences that a launch takes, at most N, their tiles numbered one after the other.
template <int N>
struct TileSpan {
    int ntok[N];
    int first[N];   // first tile of each (none: beyond all tiles)
    int tiles;      // of all
};
// Distances in bytes from the first sub-sequence's buffer to the others'. (Buffers come as a pointer to the first and these:
// pointers in a struct argument are not taken to point into global memory, and flat loads make the reduction of 16 heads x
// 32768 tokens take 54 us instead of 47.)
template <int N>
struct Distances {
    long long at[N];
};
template <int N>
DEVI int shard_of(const TileSpan<N> &sp, int t) {
    int s = 0;
#pragma unroll
    for (int i = 1; i < N; ++i) s += t >= sp.first[i];
    return s;
}
// a[s] by uniform selects (an argument indexed at run time would go through memory)
template <int N, typename V>
DEVI V pick(const V (&a)[N], int s) {
    V v = a[0];
#pragma unroll
    for (int i = 1; i < N; ++i)
        if (s >= i) v = a[i];
    return v;
}
// Where tile t lies: its sub-sequence, rows that exist, first element in a buffer [chain][token][D].
template <int N, int CT, int D>
struct Place {
    int shard, nvalid;
    size_t off;
    DEVI Place(const TileSpan<N> &sp, int chain, int t) : shard(shard_of(sp, t)) {
        const int ntok = pick(sp.ntok, shard), lt = t - pick(sp.first, shard);
        nvalid = min(CT, ntok - lt * CT);
        off = ((size_t)chain * ntok + (size_t)lt * CT) * D;
    }
    template <typename P>
    DEVI P *in(P *p, const Distances<N> &d) const {
        if constexpr (N > 1) p = (P *)((char *)p + pick(d.at, shard));
        return p + off;
    }
};

// The wave's column block of S_eff = S or S^T ([D][D] float, row-major) as MFMA operand fragments.
template <typename T, int D>
DEVI void load_fragments(const Lane &ln, typename Elem<T>::frag (&sf)[D / 32][Elem<T>::NSUB], const float *S, bool trans, int w) {
    f32x16 st[D / 32];
    if (trans) state_load_t_w<D>(ln, st, S, w);
    else state_load_w<D>(ln, st, S, w);
#pragma unroll
    for (int ab = 0; ab < D / 32; ++ab)
#pragma unroll
        for (int m = 0; m < Elem<T>::NSUB; ++m) sf[ab][m] = Elem<T>::from_acc(st[ab], m);
}
// Row stride of an output tile in LDS, rows padded by 16 bytes.
template <typename T, int D>
constexpr int out_ld() { return D + 16 / (int)sizeof(T); }
// Out = X S_eff of the tile in sX, into sO: OutT[c][i] = sum_a S_eff[a][c] X[i][a] (a taken in accumulator order).
// The accumulators hold the transposed tile (lane = token, four consecutive features per register
// group). Written to memory as they are, a store instruction would touch 32 rows with 8 or 16 bytes
// each; through LDS every row leaves as whole 16-byte pieces of consecutive lanes.
template <typename T, int CT, int D>
DEVI void product_tile(const Lane &ln, const typename Elem<T>::frag (&sf)[D / 32][Elem<T>::NSUB], const T *sX, T *sO, int w) {
    using E = Elem<T>;
    constexpr int NB = CT / 32, LDD = tile_ld<T, D>(), LDO = out_ld<T, D>();
    f32x16 acc[NB];
#pragma unroll
    for (int ib = 0; ib < NB; ++ib) acc[ib] = f32x16{0};
#pragma unroll
    for (int ab = 0; ab < D / 32; ++ab)
#pragma unroll
        for (int m = 0; m < E::NSUB; ++m)
#pragma unroll
            for (int ib = 0; ib < NB; ++ib) acc[ib] = E::mfma(sf[ab][m], E::ld_kp(ln, sX, LDD, 32 * ib, 32 * ab, m), acc[ib]);
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            E::st4(sO + (32 * ib + ln.r) * LDO + 32 * w + 8 * g + 4 * ln.h, acc[ib][4 * g], acc[ib][4 * g + 1],
                   acc[ib][4 * g + 2], acc[ib][4 * g + 3]);
}
// The output tile in sO to memory, whole rows.
template <typename T, int CT, int D, int NT>
DEVI void write_tile(T *o, const T *sO, int nrows) {
    using M = TileMover<T, CT, D, NT>;
    constexpr int LDO = out_ld<T, D>();
    const int row0 = threadIdx.x / M::VPR;
    const unsigned glo = M::lane_off(D) * sizeof(T);
    const T *src = sO + M::lane_off(LDO);
#pragma unroll
    for (int i = 0; i < M::NV; ++i)
        if (row0 + i * (NT / M::VPR) < nrows) gstore<u32x4>(o + i * (NT / M::VPR) * D, glo, *(const u32x4 *)(src + i * (NT / M::VPR) * LDO));
}

// ---------------------------------------------------------------------------
// k_bidir_reduce: partial state of one segment of one head,
//   part[chain][seg] = sum over the segment's tokens s of x_s y_s^T   ([a][c], a indexes x).
// A segment is a run of tiles over all sub-sequences of the launch. Rows past the end of a sub-sequence read as zero.
// DQ (x = Q, y = dO): also dQ = dO KV^T of every tile, KV being known from the forward pass, so that dO is read once:
// 16 heads x 32768 tokens, bf16 d=128, both passes 337 -> 316 us. At the traffic's rate: 400 MiB in 76 - 86 us.
// ---------------------------------------------------------------------------
template <typename T, int CT, int D, bool DQ, int N>
__global__ __launch_bounds__(D * 2, 2) void k_bidir_reduce(const T *__restrict__ X, const T *__restrict__ Y, float *__restrict__ part,
                                                         TileSpan<N> sp, Distances<N> dx, Distances<N> dy, int nseg, int tiles_per_seg,
                                                         T *__restrict__ dQ, Distances<N> ddq, const float *__restrict__ kv) {
    using E = Elem<T>;
    constexpr int NT = D * 2, LDD = tile_ld<T, D>(), DB = D / 32, NKS = CT / E::KSTEP;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    T *sX = (T *)smem;
    T *sY = sX + CT * LDD;
    [[maybe_unused]] T *sO = sY + CT * LDD;

    const int chain = blockIdx.y, seg = blockIdx.x;
    const int t0 = seg * tiles_per_seg;
    const int t1 = min(t0 + tiles_per_seg, sp.tiles);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave index, scalar
    Lane ln = fresh_lane();
    // Two tiles are in flight at any time: a streaming sum has nothing else to hide the memory latency with.
    TileMover<T, CT, D, NT, true> mx[2], my[2];   // streaming (non-temporal) loads
    auto request = [&](int b, int t) {
        if (t < t1) {
            const Place<N, CT, D> at(sp, chain, t);
            mx[b].load(at.in(X, dx), at.nvalid);
            my[b].load(at.in(Y, dy), at.nvalid);
        }
    };
    request(0, t0);
    request(1, t0 + 1);
    f32x16 st[DB];
#pragma unroll
    for (int ab = 0; ab < DB; ++ab) st[ab] = f32x16{0};
    typename E::frag sf[DB][E::NSUB];
    if constexpr (DQ) load_fragments<T, D>(ln, sf, kv + (size_t)chain * D * D, true, w);

    auto consume = [&](int b, int t) {
        __syncthreads();  // previous tile fully consumed
        ln = fresh_lane();
        mx[b].store(sX, LDD);
        my[b].store(sY, LDD);
        __syncthreads();
        request(b, t + 2);
        struct Step {
            typename E::frag y;
            typename E::frag x[DB];
        };
        pipelined<NKS>(
            [&](int ks) {
                Step f;
                f.y = E::ld_ks(ln, sY, LDD, ks * E::KSTEP, 32 * w);
#pragma unroll
                for (int ab = 0; ab < DB; ++ab) f.x[ab] = E::ld_ks(ln, sX, LDD, ks * E::KSTEP, 32 * ab);
                return f;
            },
            [&](int, const Step &f) {
#pragma unroll
                for (int ab = 0; ab < DB; ++ab) st[ab] = E::mfma(f.x[ab], f.y, st[ab]);
            });
        if constexpr (DQ) {
            product_tile<T, CT, D>(ln, sf, sY, sO, w);
            __syncthreads();
            const Place<N, CT, D> at(sp, chain, t);
            write_tile<T, CT, D, NT>(at.in(dQ, ddq), sO, at.nvalid);
        }
    };
    for (int t = t0; t < t1; t += 2) {
        consume(0, t);
        if (t + 1 < t1) consume(1, t + 1);
    }
    state_store_w<D>(ln, st, part + ((size_t)chain * nseg + seg) * D * D, w);
}

// state[chain] = (accumulate ? state[chain] : 0) + part[chain][0] + part[chain][1] + ..., in that order.
__global__ __launch_bounds__(256) void k_bidir_sum(const float *__restrict__ part, float *__restrict__ state, int DD, int nseg,
                                                   int accumulate) {
    const int chain = blockIdx.y;
    const int e = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (e >= DD) return;
    float *dst = state + (size_t)chain * DD + e;
    const float *src = part + (size_t)chain * nseg * DD + e;
    f32x4 acc = accumulate ? *(const f32x4 *)dst : f32x4{0, 0, 0, 0};
    constexpr int U = 8;  // partial sums fetched together (independent loads)
    for (int n0 = 0; n0 < nseg; n0 += U) {
        f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = n0 + u < nseg ? *(const f32x4 *)(src + (size_t)(n0 + u) * DD) : f32x4{0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < U; ++u) acc += v[u];
    }
    *(f32x4 *)dst = acc;
}

// ---------------------------------------------------------------------------
// k_bidir_apply: blockIdx.z selects one of up to three products Out = X S_eff,
// S_eff = S or S^T ([D][D] float per head, row-major). The wave's column block
// of S_eff is loaded once, converted to MFMA operand fragments, and kept in
// registers for every tile of the block's range (over all sub-sequences of the launch).
// ---------------------------------------------------------------------------
template <int N>
struct Ops {
    const void *x[3];
    const float *s[3];
    void *out[3];
    int trans[3];
    Distances<N> dx[3], dout[3];
};
template <typename T, int CT, int D, int N>
__global__ __launch_bounds__(D * 2, 2) void k_bidir_apply(Ops<N> ops, TileSpan<N> sp, int tiles_per_blk) {
    using E = Elem<T>;
    constexpr int NT = D * 2, LDD = tile_ld<T, D>(), DB = D / 32;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    T *sX = (T *)smem;
    T *sO = sX + CT * LDD;   // output tile [token][feature]

    const int chain = blockIdx.y, op = blockIdx.z;
    const int t0 = blockIdx.x * tiles_per_blk;
    const int t1 = min(t0 + tiles_per_blk, sp.tiles);
    if (t0 >= t1) return;  // uniform over the workgroup
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Lane ln = fresh_lane();
    const T *X = (const T *)pick(ops.x, op);
    T *O = (T *)pick(ops.out, op);
    const float *S = pick(ops.s, op) + (size_t)chain * D * D;
    const int trans = pick(ops.trans, op);
    const Distances<N> dx = pick(ops.dx, op), dout = pick(ops.dout, op);
    // Two tiles are in flight at any time (nothing else hides the memory latency of a streaming product).
    TileMover<T, CT, D, NT> mx[2];
    auto request = [&](int b, int t) {
        if (t < t1) {
            const Place<N, CT, D> at(sp, chain, t);
            mx[b].load(at.in(X, dx), at.nvalid);
        }
    };
    request(0, t0);
    request(1, t0 + 1);

    typename E::frag sf[DB][E::NSUB];
    load_fragments<T, D>(ln, sf, S, trans, w);

    auto consume = [&](int b, int t) {
        __syncthreads();  // previous tile fully consumed: sX and sO are free
        ln = fresh_lane();
        mx[b].store(sX, LDD);
        __syncthreads();
        request(b, t + 2);
        product_tile<T, CT, D>(ln, sf, sX, sO, w);
        __syncthreads();
        const Place<N, CT, D> at(sp, chain, t);
        write_tile<T, CT, D, NT>(at.in(O, dout), sO, at.nvalid);
    };
    for (int t = t0; t < t1; t += 2) {
        consume(0, t);
        if (t + 1 < t1) consume(1, t + 1);
    }
}

// ---------------------------------------------------------------------------
// Host-side launchers. N: sub-sequences of a launch (1 or kMaxShards): launches of one carry fewer arguments and no selects.
// ---------------------------------------------------------------------------
template <int N>
static TileSpan<N> span(int n, const int *ntok, int tile) {
    TileSpan<N> sp{};
    for (int i = 0; i < N; ++i) {
        sp.ntok[i] = i < n ? ntok[i] : 0;
        sp.first[i] = i < n ? sp.tiles : 0x7fffffff;
        if (i < n) sp.tiles += (ntok[i] + tile - 1) / tile;
    }
    return sp;
}
template <int N, typename V>
static Distances<N> distances(V *const *list, int n) {
    Distances<N> d{};
    for (int i = 1; list && i < n; ++i) d.at[i] = (const char *)list[i] - (const char *)list[0];
    return d;
}

template <typename T, int CT, int D, int N>
static hipError_t run_bidir_state(const BidirPlan &p, const BidirSums &a, hipStream_t s, const KernelEvents *ke) {
    const int chains = p.B * p.H, DD = D * D;
    constexpr size_t lds = (2 * (size_t)CT * tile_ld<T, D>()) * sizeof(T), lds_dq = lds + (size_t)CT * out_ld<T, D>() * sizeof(T);
    static_assert(lds_dq <= 65536, "fits the default dynamic LDS limit");
    const auto sp = span<N>(a.n, a.ntok, CT);
    if (ke) (void)hipEventRecord(ke->ev[0], s);
    const auto kernel = a.dq ? k_bidir_reduce<T, CT, D, true, N> : k_bidir_reduce<T, CT, D, false, N>;
    kernel<<<dim3(p.nseg, chains), dim3(D * 2), a.dq ? lds_dq : lds, s>>>(
        (const T *)a.x[0], (const T *)a.y[0], a.part, sp, distances<N>(a.x, a.n), distances<N>(a.y, a.n), p.nseg, p.tiles_per_seg,
        a.dq ? (T *)a.dq[0] : nullptr, distances<N>(a.dq, a.n), a.kv);
    if (ke) (void)hipEventRecord(ke->ev[1], s);
    k_bidir_sum<<<dim3((DD / 4 + 255) / 256, chains), dim3(256), 0, s>>>(a.part, a.state, DD, p.nseg, a.accumulate);
    if (ke) {
        (void)hipEventRecord(ke->ev[2], s);
        (void)hipEventRecord(ke->ev[3], s);
    }
    return hipGetLastError();
}

template <typename T, int CT, int D, int N>
static hipError_t run_bidir_apply(const BidirPlan &p, const BidirProducts &a, hipStream_t s, const KernelEvents *ke) {
    const int chains = p.B * p.H;
    constexpr size_t lds = (size_t)CT * (tile_ld<T, D>() + out_ld<T, D>()) * sizeof(T);
    static_assert(2 * lds <= 163840, "two workgroups per CU");
    if (hipError_t e = allow_dynamic_lds((const void *)k_bidir_apply<T, CT, D, N>, lds); e != hipSuccess) return e;
    const auto sp = span<N>(a.n, a.ntok, CT);
    Ops<N> ops{};
    for (int i = 0; i < a.nops; ++i) {
        ops.x[i] = a.x[i][0];
        ops.s[i] = a.s[i];
        ops.out[i] = a.out[i][0];
        ops.trans[i] = a.trans[i];
        ops.dx[i] = distances<N>(a.x[i], a.n);
        ops.dout[i] = distances<N>(a.out[i], a.n);
    }
    const lasp::Blocks blk = blocks_for(sp.tiles, (long long)chains * a.nops, kBidirTargetWorkgroups);
    if (ke) {
        (void)hipEventRecord(ke->ev[0], s);
        (void)hipEventRecord(ke->ev[1], s);
        (void)hipEventRecord(ke->ev[2], s);
    }
    k_bidir_apply<T, CT, D, N><<<dim3(blk.count, chains, a.nops), dim3(D * 2), lds, s>>>(ops, sp, blk.tiles);
    if (ke) (void)hipEventRecord(ke->ev[3], s);
    return hipGetLastError();
}

int bidir_reduce_tile(int dtype) { return dtype == 0 ? 32 : 64; }

template <int N>
static hipError_t sums_of(const BidirPlan &p, const BidirSums &a, hipStream_t s, const KernelEvents *ke) {
    if (p.dtype == 0) return p.D == 64 ? run_bidir_state<float, 32, 64, N>(p, a, s, ke) : run_bidir_state<float, 32, 128, N>(p, a, s, ke);
    return p.D == 64 ? run_bidir_state<bf16_t, 64, 64, N>(p, a, s, ke) : run_bidir_state<bf16_t, 64, 128, N>(p, a, s, ke);
}
hipError_t launch_bidir_sums(const BidirPlan &p, const BidirSums &a, hipStream_t s, const KernelEvents *ke) {
    return a.n == 1 ? sums_of<1>(p, a, s, ke) : sums_of<kMaxShards>(p, a, s, ke);
}
hipError_t launch_bidir_state(const BidirPlan &p, const void *x, const void *y, float *state, int accumulate, float *part,
                              hipStream_t stream, const KernelEvents *ke) {
    return launch_bidir_sums(p, BidirSums{1, &p.N, &x, &y, state, accumulate, part, nullptr, nullptr}, stream, ke);
}

// The apply pass keeps no state between tiles, so it reads long tiles: 128 tokens of bfloat16,
// 64 of float (more bytes in flight per workgroup, fewer barriers).
int bidir_product_tile(int dtype) { return dtype == 0 ? 64 : 128; }

template <int N>
static hipError_t products_of(const BidirPlan &p, const BidirProducts &a, hipStream_t s, const KernelEvents *ke) {
    if (p.dtype == 0) return p.D == 64 ? run_bidir_apply<float, 64, 64, N>(p, a, s, ke) : run_bidir_apply<float, 64, 128, N>(p, a, s, ke);
    return p.D == 64 ? run_bidir_apply<bf16_t, 128, 64, N>(p, a, s, ke) : run_bidir_apply<bf16_t, 128, 128, N>(p, a, s, ke);
}
hipError_t launch_bidir_products(const BidirPlan &p, const BidirProducts &a, hipStream_t s, const KernelEvents *ke) {
    return a.n == 1 ? products_of<1>(p, a, s, ke) : products_of<kMaxShards>(p, a, s, ke);
}
hipError_t launch_bidir_apply(const BidirPlan &p, const BidirOps &ops, int nops, hipStream_t stream, const KernelEvents *ke) {
    BidirProducts a{1, &p.N, nops, {}, {}, {}, {}};
    for (int i = 0; i < nops; ++i) {
        a.x[i] = &ops.x[i];
        a.s[i] = ops.s[i];
        a.out[i] = &ops.out[i];
        a.trans[i] = ops.trans[i];
    }
    return launch_bidir_products(p, a, stream, ke);
}

}  // namespace lasp
