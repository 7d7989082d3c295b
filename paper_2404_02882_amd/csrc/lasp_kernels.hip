// HIP kernels (gfx950 / CDNA4) that do not depend on the data type's tiles: the scan over segment states, the gradient
// of the per-token log decay, the sum over grouped heads, the library's fixed scratch; and the dispatch to the
// walks (lasp_walks.hip) by data type and dimensions.
#include <hip/hip_runtime.h>

#include <mutex>

#include "lasp_internal.h"
#include "lasp_rules.h"
#include "lasp_device.h"

namespace lasp {

// ---------------------------------------------------------------------------
// k_scan: per state element, scan over the segments of a head.
//   forward : start_0 = kv_in (or 0); start_{j+1} = lambda^(len_j) start_j + local_j
//   backward: recv_{S-1} = dkv_out (or 0); recv_{j-1} = lambda^(len_j) recv_j + local_j
// scratch[chain][j] ([d_k][d_v] floats each) holds local_j on entry and start_j / recv_j on exit.
// ---------------------------------------------------------------------------
// With per-token decay the factor of segment j is 2^seglog[chain][j] (written by k_local).
// SHARED: over the segments of several sub-sequences (nslots), counting where each ends. In launches of one that counting took
// the scan over 87 segments of one head from 12.2 to 13.3 us, over 33 of 16 heads, d=64, from 6.0 to 6.5: its own instance.
// U: segments whose local states are fetched together. The scan is a chain of as many waits for memory as it has such batches,
// but a batch costs its whole length, and where many states are scanned their loads are in flight side by side anyway. Steps with
// 8 / 16 / 32, us: 2 heads x 32768 tokens (128 segments) 117.8 / 115.1 / 111.3, 2 x 6031 (48) 61.0 / 59.8 / 60.3, 2 x 1280 (10) 42.1 / 41.7 / 43.0,
// d=64 8 x 8192 (64) 58.6 / 57.2 / 56.4; 16 x 2048 (16) 73.8 / 74.8 / 75.8; float 1 x 1400 (44) 61.2 / 60.2 / 60.5, 8 x 895 x 4 (112, twice the
// states) 213.4 / 213.2 / 214.6. With a decay per token, whose factors are computed, long batches pay later: 2 x 2300 (18) 56.0 / 56.5 /
// 56.8, 2 x 2080 (33) 50.7 / 50.8 / 53.5, 2 x 16384 (128) 109.2 / 106.4 / 106.6.
template <bool BWD, bool TOKEN, bool SHARED, int U>
__global__ __launch_bounds__(256) void k_scan(float *__restrict__ scratch, const float *__restrict__ boundary,
                                              const float *__restrict__ decay, const float *__restrict__ seglog,
                                              int H, int DD, int nseg, int slots, int seg_tokens, int ntok) {
    const int chain = blockIdx.y, nslots = SHARED ? slots : nseg;
    const int e = (blockIdx.x * blockDim.x + threadIdx.x) * 4;  // four consecutive state elements per thread
    if (e >= DD) return;
    const SegDecay<TOKEN> seg_decay(decay, TOKEN ? seglog + (size_t)chain * nslots : nullptr, chain, H, nseg, seg_tokens, ntok);
    // The caller's state and the segment states share one layout, [d_k][d_v] (DD = d_k * d_v elements).
    f32x4 carry = {0, 0, 0, 0};
    if (boundary) carry = *(const f32x4 *)(boundary + (size_t)chain * DD + e);
    float *s = scratch + (size_t)chain * nslots * DD + e;
    ShardEnds<BWD, SHARED> ends(nseg);
    for (int n0 = 0; n0 < nslots; n0 += U) {
        f32x4 local[U];
        float factor[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n = n0 + u, j = BWD ? nslots - 1 - n : n;
            const bool has_local = n < nslots && (BWD ? (j > 0) : (j < nslots - 1));
            local[u] = has_local ? *(const f32x4 *)(s + (size_t)j * DD) : f32x4{0, 0, 0, 0};
            const bool end = ends.next(j);
            factor[u] = !TOKEN || has_local ? seg_decay(j, end) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int n = n0 + u, j = BWD ? nslots - 1 - n : n;
            if (n < nslots) {
                *(f32x4 *)(s + (size_t)j * DD) = carry;
                carry = factor[u] * carry + local[u];
            }
        }
    }
}

hipError_t launch_scan(const Plan &p, bool bwd, float *states, const float *boundary, const float *decay, const float *seglog,
                       hipStream_t s) {
    const int DD = p.dk * p.dv, nslots = p.shards * p.nseg;   // states hold the real rows and columns only
    const dim3 grid((DD / 4 + 255) / 256, p.B * p.H);
    const auto of = [&](auto u) {
        constexpr int U = decltype(u)::value;
        return p.shards > 1 ? (bwd ? k_scan<true, false, true, U> : k_scan<false, false, true, U>)
               : bwd        ? (p.token ? k_scan<true, true, false, U> : k_scan<true, false, false, U>)
                            : (p.token ? k_scan<false, true, false, U> : k_scan<false, false, false, U>);
    };
    const bool few_states = (long long)p.B * p.H * DD <= 65536;   // of four heads at d = 128, 16 at d = 64
    const auto kernel = nslots <= (p.token ? 22 : 16)               ? of(std::integral_constant<int, 8>{})
                        : !p.token && nslots >= 48 && few_states ? of(std::integral_constant<int, 32>{}) : of(std::integral_constant<int, 16>{});
    kernel<<<grid, dim3(256), 0, s>>>(states, boundary, p.token ? nullptr : decay, seglog, p.H, DD, p.nseg, nslots,
                                      p.tiles_per_seg * p.tile, p.N);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// k_dlg: gradient of the per-token log decay from r_t = q_t.dq_t - k_t.dk_t
// (written per tile by the backward walk):
//     dlog g_s = <dkv_out, kv_out> + sum_{t >= s} r_t.
// It follows from expanding <D_s, kv_s> with either recurrence, kv_s = g_s kv_{s-1}
// + k_s v_s^T or D_s = q_s do_s^T + g_{s+1} D_{s+1} (D_s: gradient w.r.t. kv_s):
// dlog g_s + k_s.dk_s = q_s.dq_s + dlog g_{s+1}. One workgroup per block of
// kDlgBlock tokens of a head: it sums everything behind its block (r of the later
// tokens and the boundary term), then scans its own tokens from the right. Sums
// are carried in double; the order of additions is fixed, so reruns are identical.
// ---------------------------------------------------------------------------
constexpr int kDlgBlock = 1024;  // tokens per workgroup: 256 threads x 4

DEVI double block_sum(double x, double *sh) {  // sum over the 256 threads, returned to all
    const int tid = threadIdx.x;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    __syncthreads();
    if ((tid & 63) == 0) sh[tid >> 6] = x;
    __syncthreads();
    return sh[0] + sh[1] + sh[2] + sh[3];
}

__global__ __launch_bounds__(256) void k_dlg(const float *__restrict__ rtok, const float *__restrict__ kv_out,
                                             const float *__restrict__ dkv_out, float *__restrict__ dlg, int N, int DD) {
    __shared__ double sh[4];
    const int chain = blockIdx.y, tid = threadIdx.x;
    const int s0 = blockIdx.x * kDlgBlock;  // first token of this block
    const float *r = rtok + (size_t)chain * N;
    double behind = 0.0;
    if (dkv_out) {
        const f32x4 *a = (const f32x4 *)(kv_out + (size_t)chain * DD), *b = (const f32x4 *)(dkv_out + (size_t)chain * DD);
        for (int e = tid; e < DD / 4; e += 256) {
            const f32x4 x = a[e], y = b[e];
            behind += (double)x[0] * y[0] + (double)x[1] * y[1] + (double)x[2] * y[2] + (double)x[3] * y[3];
        }
    }
    if (N % 4 == 0) {   // rows of r are 16-byte aligned: four tokens per load, four loads in flight
        double b1 = 0.0, b2 = 0.0, b3 = 0.0;
        int s = s0 + kDlgBlock + 4 * tid;
        for (; s + 3 * kDlgBlock < N; s += 4 * kDlgBlock) {
            const f32x4 x0 = *(const f32x4 *)(r + s), x1 = *(const f32x4 *)(r + s + kDlgBlock),
                        x2 = *(const f32x4 *)(r + s + 2 * kDlgBlock), x3 = *(const f32x4 *)(r + s + 3 * kDlgBlock);
            behind += ((double)x0[0] + x0[1]) + ((double)x0[2] + x0[3]);
            b1 += ((double)x1[0] + x1[1]) + ((double)x1[2] + x1[3]);
            b2 += ((double)x2[0] + x2[1]) + ((double)x2[2] + x2[3]);
            b3 += ((double)x3[0] + x3[1]) + ((double)x3[2] + x3[3]);
        }
        for (; s < N; s += kDlgBlock) {
            const f32x4 x = *(const f32x4 *)(r + s);
            behind += ((double)x[0] + x[1]) + ((double)x[2] + x[3]);
        }
        behind += (b1 + b2) + b3;
    } else {
        for (int s = s0 + kDlgBlock + tid; s < N; s += 256) behind += (double)r[s];
    }
    behind = block_sum(behind, sh);
    // this thread's four tokens, suffix sums inside the group
    const int s = s0 + 4 * tid;
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = s + e < N ? r[s + e] : 0.0f;
    double v3 = x[3], v2 = v3 + x[2], v1 = v2 + x[1], v0 = v1 + x[0];
    // exclusive suffix sum of the group totals over the threads behind this one
    double incl = v0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double y = __shfl_down(incl, d, 64);
        if ((tid & 63) + d < 64) incl += y;
    }
    __syncthreads();
    if ((tid & 63) == 0) sh[tid >> 6] = incl;  // total of this wave
    __syncthreads();
    double after = behind + (incl - v0);
    for (int wv = (tid >> 6) + 1; wv < 4; ++wv) after += sh[wv];
    const double v[4] = {v0, v1, v2, v3};
    float *o = dlg + (size_t)chain * N;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (s + e < N) o[s + e] = (float)(after + v[e]);
}

hipError_t launch_dlg(const Plan &p, const BwdArgs &a, hipStream_t s) {
    k_dlg<<<dim3((p.N + kDlgBlock - 1) / kDlgBlock, p.B * p.H), dim3(256), 0, s>>>(a.rtok, a.kv_out, a.dkv_out, a.dlog_g, p.N, p.dk * p.dv);
    return hipGetLastError();
}

// Grouped K/V heads, backward: the walking kernel wrote dK, dV per QUERY head into `part`
// ([chains][ntok][D], in the data type, so each partial gradient is already rounded to it once);
// dK, dV of a K/V head are the sums over its kvdiv query heads, added in fp32 in a fixed order and
// rounded to the data type a second time. For bfloat16 the partials' rounding errors (2^-9 relative
// each, independent) add in quadrature, so the sum stays well inside the 2e-2 bound also for
// multi-query attention (tested with 16 query heads per K/V head).
// Bound by the parts' traffic: a thread takes 16 bytes of every part, the parts of four heads in flight at once. 32 heads x
// 8192 tokens, d=128, four K/V heads (134 MB of parts): 30.2 -> 24.7 us against single
// values of one part after the other.
template <typename T>
__global__ __launch_bounds__(256) void k_group_sum(const T *__restrict__ dk_part, const T *__restrict__ dv_part, GroupOut out, int kvdiv,
                                                   size_t dk_head, size_t dv_head) {
    constexpr int V = 16 / sizeof(T), U = 4;   // values of a piece, pieces in flight
    const int shard = blockIdx.z >> 1;
    const bool values = blockIdx.z & 1;
    const size_t kvchain = blockIdx.y, per_head = values ? dv_head : dk_head;   // ntok * D: whole pieces
    const T *src = (values ? dv_part : dk_part) + (shard * gridDim.y + kvchain) * kvdiv * per_head;
    T *dst = (T *)(values ? out.dv[shard] : out.dk[shard]) + kvchain * per_head;
    for (size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * V; e < per_head; e += (size_t)gridDim.x * 256 * V) {
        float acc[V] = {};
        for (int g0 = 0; g0 < kvdiv; g0 += U) {
            u32x4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (g0 + u < kvdiv) x[u] = *(const u32x4 *)(src + (size_t)(g0 + u) * per_head + e);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (g0 + u >= kvdiv) break;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (sizeof(T) == 2) {
                        acc[2 * i] += __uint_as_float(x[u][i] << 16);
                        acc[2 * i + 1] += __uint_as_float(x[u][i] & 0xffff0000u);
                    } else {
                        acc[i] += __uint_as_float(x[u][i]);
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < V; i += 4) Elem<T>::st4(dst + e + i, acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
    }
}
template <typename T>
static hipError_t run_group_sum(const Plan &p, const BwdArgs &a, hipStream_t s) {
    const size_t dk_head = (size_t)p.N * p.dk, dv_head = (size_t)p.N * p.dv;
    const int kvchains = p.B * (p.H / p.kvdiv);
    size_t blocks = ((dk_head > dv_head ? dk_head : dv_head) * sizeof(T) / 16 + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    k_group_sum<T><<<dim3((unsigned)blocks, kvchains, 2 * p.shards), dim3(256), 0, s>>>((const T *)a.dk, (const T *)a.dv, a.group, p.kvdiv,
                                                                                     dk_head, dv_head);
    return hipGetLastError();
}

hipError_t launch_group_sum(const Plan &p, const BwdArgs &a, hipStream_t s) {
    return p.dtype == 0 ? run_group_sum<float>(p, a, s) : run_group_sum<bf16_t>(p, a, s);
}

// Scratch of the entry point that allocates nothing (lasp_fwd_noalloc): the segment states live in this
// array instead of a buffer the caller brings. Every device the library runs on holds its own copy, at
// its own address, until the process ends. The name below is a host-side stand-in, not a device address:
// host code uses the pointer static_scratch() returns, never the name.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch(void **ptr) {
    static std::mutex mu;
    static void *addr[64] = {};   // per device, filled on the first call with that device current
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> hold(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        if (hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)); e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

// Tokens per kernel tile: 32 for float data, 64 for bfloat16 data, whatever the
// chunk (both divide every supported chunk length). 64-token bfloat16 tiles let two
// forward workgroups, or one backward workgroup with every tile it needs, live on a CU.
int tile_tokens(int dtype, int chunk, int D) {
    (void)chunk;
    (void)D;
    return dtype == 0 ? 32 : 64;
}

// ---------------------------------------------------------------------------
// k_step: forward of a few tokens onto a carried state (generation), by the token recurrence itself:
//     kv_s = g_s kv_{s-1} + k_s v_s^T,   out_s = kv_s^T q_s     (fp32, on the vector units)
// A call of N <= kStepTokens tokens is bound by the state's way in and out (64 KB each per head at d=128) and by
// latency; the tile walk spends a whole 64-token tile on it. One workgroup per head and 32 value columns: thread
// (row, 4 columns) keeps DK / 32 state rows in registers, so the state is read and written once, in 128-byte row
// segments, whatever N is. Beside it a token costs R fused multiply-adds of four for the update and as many for the
// output, and one reduction over the rows. 128 heads, d=128, bf16: the walk 9.3 us at any N up to 64; this kernel
// 4.6 us at N = 1, 5.5 at 4, 7.1 at 8, 8.9 at 12, 10.5 at 16 (float: walk 12.5; d=64: walk 6.4, this 6.0 at 12): the line
// is drawn at 12. Calls that keep a state cache or normalise stay with the walk.
// ---------------------------------------------------------------------------
constexpr int kStepTokens = 12;
template <typename T, int DK, bool TOKEN>
__global__ __launch_bounds__(256) void k_step(const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V,
                                              const float *__restrict__ kv_in, const float *__restrict__ decay, T *__restrict__ O,
                                              float *__restrict__ kv_out, float *__restrict__ kv_copy, int H, int ntok, int dv, int kvdiv) {
    constexpr int R = DK / 32;
    __shared__ float sq[kStepTokens][DK], sk[kStepTokens][DK];
    __shared__ __attribute__((aligned(16))) float sv[kStepTokens][32], red[kStepTokens][4][32];
    __shared__ float sg[kStepTokens];
    const int chain = blockIdx.y, c0 = 32 * blockIdx.x, tid = threadIdx.x;
    const int kvchain = (chain / H) * (H / kvdiv) + (chain % H) / kvdiv;   // this head's K, V
    const int row = tid >> 3, col = 4 * (tid & 7);
    f32x4 st[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
        st[r] = kv_in ? *(const f32x4 *)(kv_in + ((size_t)chain * DK + row + 32 * r) * dv + c0 + col) : f32x4{0, 0, 0, 0};
    if (kv_copy) {
#pragma unroll
        for (int r = 0; r < R; ++r) *(f32x4 *)(kv_copy + ((size_t)chain * DK + row + 32 * r) * dv + c0 + col) = st[r];
    }
    for (int i = tid; i < ntok * DK; i += 256) {
        sq[i / DK][i % DK] = Elem<T>::ld1(Q + (size_t)chain * ntok * DK + i);
        sk[i / DK][i % DK] = Elem<T>::ld1(K + (size_t)kvchain * ntok * DK + i);
    }
    for (int i = tid; i < ntok * 32; i += 256) sv[i / 32][i % 32] = Elem<T>::ld1(V + ((size_t)kvchain * ntok + i / 32) * dv + c0 + i % 32);
    if (tid < ntok) sg[tid] = TOKEN ? expf(decay[(size_t)chain * ntok + tid]) : decay[chain % H];
    __syncthreads();
    for (int s = 0; s < ntok; ++s) {
        const f32x4 v = *(const f32x4 *)&sv[s][col];
        const float g = sg[s];
        f32x4 o = {0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            st[r] = g * st[r] + sk[s][row + 32 * r] * v;
            o += sq[s][row + 32 * r] * st[r];
        }
        // over the wave's eight rows (lanes 8 apart), then over the waves through LDS
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(o[e]), 0x128, 0xf, 0xf, false));   // row_ror:8
            o[e] += __shfl_xor(o[e], 16, 64);
            o[e] = add_other_half(o[e]);
        }
        if ((tid & 63) < 8) *(f32x4 *)&red[s][tid >> 6][col] = o;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) *(f32x4 *)(kv_out + ((size_t)chain * DK + row + 32 * r) * dv + c0 + col) = st[r];
    __syncthreads();
    for (int i = tid; i < ntok * 32; i += 256) {
        const int s = i / 32, c = i % 32;
        Elem<T>::st1(O + ((size_t)chain * ntok + s) * dv + c0 + c, (red[s][0][c] + red[s][1][c]) + (red[s][2][c] + red[s][3][c]));
    }
}
template <typename T>
static hipError_t run_step(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) {
    auto kernel = p.dk == 64 ? (p.token ? k_step<T, 64, true> : k_step<T, 64, false>) : (p.token ? k_step<T, 128, true> : k_step<T, 128, false>);
    if (ke)
        for (int i = 0; i < 3; ++i) (void)hipEventRecord(ke->ev[i], s);
    kernel<<<dim3(p.dv / 32, p.B * p.H), dim3(256), 0, s>>>((const T *)a.q, (const T *)a.k, (const T *)a.v, a.kv_in, a.decay, (T *)a.out,
                                                          a.kv_out, a.kv_copy, p.H, p.N, p.dv, p.kvdiv);
    if (ke) (void)hipEventRecord(ke->ev[3], s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// k_short: forward of a short float sequence (a prompt; no cache, one lambda per head) as its definition, without states between
// tiles: the workgroup of 32 queries takes the score product with every 32 keys before them on a wave of its own,
//     out_i = sum_{j <= i} lambda^(i-j) (q_i . k_j) v_j + lambda^(i+1) KV_in^T q_i,
// and d/32 more workgroups a head each sum 32 columns of kv_out, a wave for 32 tokens. Nothing goes through LDS but the
// waves' sums: a lane loads its MFMA operands from memory and splits them itself (the scores' accumulators are the other
// operand of the product with V as they are). Such a call is all latency: local pass, scan and walk one behind the other.
// Float weights reach over a tile at most, from tile to tile the sums decay, and the state's weight is a double: lambda^245 may be
// below the smallest float, and an infinity would meet that zero. (Two floats for lambda^32, whose rounded seventh power is 1e-7 off.)
// Bound by the splits of a wave's operands and the way to memory and back. 2 heads x 256 tokens, d=64, 14.1 -> 10.1 us, x 128
// 11.9 -> 7.0, x 64 8.6 -> 6.3 (the call through the Python binding takes 6); d=128 16 x 256 26.8 -> 16.9, with a state 26.7 -> 22.8.
// Error against 64 bits, the walks / this, out and kv_out: 2 x 256, d=64, 1.56e-7, 1.02e-7 / 1.00e-7, 6.9e-8; 16 x 13 1.02e-7, 3.7e-8 /
// 6.6e-8, 3.4e-8; d=128 with a state 16 x 250 2.07e-7, 1.58e-7 / 1.65e-7, 2.7e-8.
// ---------------------------------------------------------------------------
constexpr int kShortTokens = 256, kShortWaves = kShortTokens / 32;
template <int D>
__global__ __launch_bounds__(64 * kShortWaves) void k_short(const float *__restrict__ Q, const float *__restrict__ K, const float *__restrict__ V,
                                                            const float *__restrict__ kv_in, const float *__restrict__ decay,
                                                            float *__restrict__ O, float *__restrict__ kv_out, float *__restrict__ kv_copy,
                                                            int H, int ntok, int kvdiv) {
    using E = WalkElem<float>;
    using F = typename E::frag;
    constexpr int DB = D / 32, PART = DB * 1024;   // floats of a wave's sums
    extern __shared__ __attribute__((aligned(16))) float sums[];
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    float *pw = sums + (kShortWaves + 1) * PART;   // (the state's part behind the waves'); lambda^0 .. lambda^32
    f32x2 *factor = (f32x2 *)(pw + 34);      // the same in two parts
    const int chain = blockIdx.y, ntiles = (ntok + 31) / 32, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Lane ln(threadIdx.x);
    const int kvchain = (chain / H) * (H / kvdiv) + (chain % H) / kvdiv;   // this head's K, V
    Q += (size_t)chain * ntok * D;
    O += (size_t)chain * ntok * D;
    K += (size_t)kvchain * ntok * D;
    V += (size_t)kvchain * ntok * D;
    const float lam = decay[chain % H];
    if (threadIdx.x <= 32) {
        const double p = pow_small(lam, threadIdx.x);
        float hi = (float)p;
        pw[threadIdx.x] = hi;
        if (hi > p) hi = __uint_as_float(__float_as_uint(hi) - 1);
        factor[threadIdx.x] = f32x2{hi, fmaxf((float)(p - hi), hi * 0x1p-60f)};   // (none zero: an infinity stays one)
    }
    auto row8 = [&](const float *x, int row, int col) {   // eight features of a token (zero past the end)
        const float *p = x + (size_t)row * D + col;
        const f32x4 z = {0, 0, 0, 0}, lo = row < ntok ? *(const f32x4 *)p : z, hi = row < ntok ? *(const f32x4 *)(p + 4) : z;
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto split = [](const f32x8 &x) { return E::template split<false>(x, nullptr); };
    f32x16 acc[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) acc[b] = f32x16{0};
    auto put = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4 *)(sums + slot * PART + ((4 * b + q) * 64 + ln.id) * 4) = f32x4{acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]};
    };
    auto part = [&](int v, int i) { return *(const f32x4 *)(sums + v * PART + 4 * i); };   // i: four values of a wave's sums
    auto decayed = [](f32x2 f, const f32x4 &x, const f32x4 &y) {   // f x + y
        f32x4 z;
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = __builtin_fmaf(f[0], x[e], __builtin_fmaf(f[1], x[e], y[e]));
        return z;
    };
    // the state's weight at the lane's query (in kv_out: at the end)
    const double up = kv_in ? fmax(pow_small(lam, (int)blockIdx.x < ntiles ? 32 * blockIdx.x + ln.r : ntok - 1) * lam, 0x1p-1000) : 0.0;
    if ((int)blockIdx.x < ntiles) {
        const int t = blockIdx.x, query = 32 * t + ln.r;
        const bool keys = w <= t, state = kv_in && w == (t + 1 < kShortWaves ? t + 1 : 0);   // what this wave has to add
        f32x16 s = {0}, low = {0};   // (the small terms apart, as in the local pass)
        f32x8 values[E::NSUB][DB];   // V, the keys in the order of the accumulator's rows
        if (keys) {
            // (requests first: a split has a branch in it, over which the compiler moves none)
            constexpr int AHEAD = 4;
#pragma unroll
            for (int k0 = 0; k0 < D / E::KSTEP; k0 += AHEAD) {
                f32x8 k[AHEAD], q[AHEAD];
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) {
                    k[i] = row8(K, 32 * w + ln.r, (k0 + i) * E::KSTEP + 8 * ln.h);
                    q[i] = row8(Q, query, (k0 + i) * E::KSTEP + 8 * ln.h);
                }
                if (k0 + AHEAD == D / E::KSTEP) {
#pragma unroll
                    for (int m = 0; m < E::NSUB; ++m)
#pragma unroll
                        for (int b = 0; b < DB; ++b)
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const int key = 32 * w + ln.acc_row(8 * m + e);
                                values[m][b][e] = key < ntok ? V[(size_t)key * D + 32 * b + ln.r] : 0.0f;
                            }
                }
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) {
                    const F kf = split(k[i]), qf = split(q[i]);
                    low = E::mfma_low(kf, qf, low);
                    s = E::mfma_high(kf, qf, s);
                }
            }
            s += low;
        }
        __syncthreads();   // the powers
        if (state) {
            const float *kv = kv_in + (size_t)chain * D * D;
            for (int ks = 0; ks < D / E::KSTEP; ++ks) {
                const f32x8 q = row8(Q, query, ks * E::KSTEP + 8 * ln.h);
                f32x8 x[DB];
#pragma unroll
                for (int b = 0; b < DB; ++b)
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[b][e] = kv[(ks * E::KSTEP + 8 * ln.h + e) * D + 32 * b + ln.r];
                const F qf = split(q);
#pragma unroll
                for (int b = 0; b < DB; ++b) acc[b] = E::mfma(split(x[b]), qf, acc[b]);
            }
            put(kShortWaves);
#pragma unroll
            for (int b = 0; b < DB; ++b) acc[b] = f32x16{0};
        }
        if (keys) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {   // to the query in its own tile, to the tile's end in those before
                const int back = (w == t ? ln.r : 31) - ln.acc_row(i);
                s[i] = back >= 0 ? s[i] * pw[back < 0 ? 0 : back] : 0.0f;
            }
#pragma unroll
            for (int m = 0; m < E::NSUB; ++m) {
                f32x8 p;
#pragma unroll
                for (int e = 0; e < 8; ++e) p[e] = s[8 * m + e];
                const F pf = split(p);
#pragma unroll
                for (int b = 0; b < DB; ++b) acc[b] = E::mfma(split(values[m][b]), pf, acc[b]);
            }
        }
        if (keys) put(w);
        __syncthreads();
        const f32x2 tile = factor[32];
        for (int i = threadIdx.x; i < PART / 4; i += 64 * kShortWaves) {
            const Lane of(i);
            const int token = 32 * t + of.r, feature = 8 * (i >> 6) + 4 * of.h;
            f32x4 x = {0, 0, 0, 0};
#pragma unroll 4   // (of one by one the waits for LDS add up: 10.17 us, so 10.04)
            for (int v = 0; v < t; ++v) x = decayed(tile, x, part(v, i));
            x = decayed(factor[of.r + 1], x, part(t, i));
            if (kv_in) {
                const f32x4 in = part(kShortWaves, i);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = (float)fma(up, (double)in[e], (double)x[e]);
            }
            if (token < ntok) *(f32x4 *)(O + (size_t)token * D + feature) = x;
        }
    } else {
        const int c = 32 * (blockIdx.x - ntiles) + ln.r;
        constexpr int NKS = 32 / E::KSTEP;
        f32x8 y[NKS], x[NKS][DB];
        if (w < ntiles) {
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int token = 32 * w + ks * E::KSTEP + 8 * ln.h + e;
                    y[ks][e] = token < ntok ? V[(size_t)token * D + c] : 0.0f;
#pragma unroll
                    for (int b = 0; b < DB; ++b) x[ks][b][e] = token < ntok ? K[(size_t)token * D + 32 * b + ln.r] : 0.0f;
                }
        }
        __syncthreads();   // the powers
        if (w < ntiles) {
            F v[NKS];
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int after = min(32, ntok - 32 * w) - 1 - (ks * E::KSTEP + 8 * ln.h + e);
                    y[ks][e] *= pw[after < 0 ? 0 : after];   // (past the end: zero times one)
                }
                v[ks] = split(y[ks]);
            }
#pragma unroll
            for (int b = 0; b < DB; ++b) {
                f32x16 low = {0};
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    const F k = split(x[ks][b]);
                    low = E::mfma_low(k, v[ks], low);
                    acc[b] = E::mfma_high(k, v[ks], acc[b]);
                }
                acc[b] += low;
            }
            put(w);
        }
        __syncthreads();
        const f32x2 tile = factor[32];
        for (int i = threadIdx.x; i < PART / 4; i += 64 * kShortWaves) {
            const Lane of(i);
            f32x4 x = {0, 0, 0, 0};
            const size_t at = ((size_t)chain * D + 8 * (i >> 6) + 4 * of.h) * D + 32 * (blockIdx.x - ntiles) + of.r;
#pragma unroll 4
            for (int v = 0; v + 1 < ntiles; ++v) x = decayed(tile, x, part(v, i));
            x = decayed(factor[ntok - 32 * (ntiles - 1)], x, part(ntiles - 1, i));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (kv_in) {
                    const float in = kv_in[at + e * D];
                    x[e] = (float)fma(up, (double)in, (double)x[e]);
                    if (kv_copy) kv_copy[at + e * D] = in;
                }
                kv_out[at + e * D] = x[e];
            }
        }
    }
}
template <int D>
static hipError_t run_short(const Plan &p, const FwdArgs &a, hipStream_t s, const KernelEvents *ke) {
    constexpr size_t lds = ((kShortWaves + 1) * D / 32 * 1024 + 3 * 34) * sizeof(float);
    static_assert(lds <= 163840, "LDS of one CU");
    if (hipError_t e = allow_dynamic_lds((const void *)k_short<D>, lds); e != hipSuccess) return e;
    if (ke)
        for (int i = 0; i < 3; ++i) (void)hipEventRecord(ke->ev[i], s);
    k_short<D><<<dim3((p.N + 31) / 32 + D / 32, p.B * p.H), dim3(64 * kShortWaves), lds, s>>>(
        (const float *)a.q, (const float *)a.k, (const float *)a.v, a.kv_in, a.decay, (float *)a.out, a.kv_out, a.kv_copy, p.H, p.N, p.kvdiv);
    if (ke) (void)hipEventRecord(ke->ev[3], s);
    return hipGetLastError();
}

// The walks by data type (float, bfloat16) and dimensions (d_k, d_v); see lasp_walks.hip.
template <typename Fn>
static Fn by_shape(const Plan &p, Fn f64, Fn f128, Fn f64_128, Fn f128_64, Fn b64, Fn b128, Fn b64_128, Fn b128_64) {
    if (p.dk != p.dv) return p.dtype == 0 ? (p.dk == 64 ? f64_128 : f128_64) : (p.dk == 64 ? b64_128 : b128_64);
    return p.dtype == 0 ? (p.D == 64 ? f64 : f128) : (p.D == 64 ? b64 : b128);
}
hipError_t launch_fwd(const Plan &p, const FwdArgs &a, hipStream_t stream, const KernelEvents *ke) {
    if (p.N <= kStepTokens && !a.cache && !p.norm && p.shards == 1) return p.dtype == 0 ? run_step<float>(p, a, stream, ke) : run_step<bf16_t>(p, a, stream, ke);
    if (p.dtype == 0 && p.dk == p.dv && !p.token && !p.norm && !a.cache && !a.states_only && p.shards == 1 && short_forward(p.N, (long long)p.B * p.H, p.D))
        return p.D == 64 ? run_short<64>(p, a, stream, ke) : run_short<128>(p, a, stream, ke);
    return by_shape(p, fwd_f32_64, fwd_f32_128, fwd_f32_64_128, fwd_f32_128_64, fwd_bf16_64, fwd_bf16_128, fwd_bf16_64_128,
                    fwd_bf16_128_64)(p, a, stream, ke);
}
hipError_t launch_bwd(const Plan &p, const BwdArgs &a, hipStream_t stream, const KernelEvents *ke) {
    return by_shape(p, bwd_f32_64, bwd_f32_128, bwd_f32_64_128, bwd_f32_128_64, bwd_bf16_64, bwd_bf16_128, bwd_bf16_64_128,
                    bwd_bf16_128_64)(p, a, stream, ke);
}

}  // namespace lasp
