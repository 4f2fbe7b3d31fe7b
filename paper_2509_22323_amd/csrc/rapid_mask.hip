// Block-mask selection for the Sparse-Attention levels, MI355X (gfx950).  C ABI and the rule:
// include/rapid_mask.h (RAPID^3 Sec. 3.2 Level-3 and Sec. 3.3 (c) describe what the mask is
// for; the rule is this library's own).
//
// Two kernels.  block_mean_kernel streams Q and K once (HBM-bound: 2 bytes per element read,
// 4 * D bytes per block written) and leaves fp32 block means in the workspace.
// select_blocks_small_kernel (up to 256 blocks per side) and select_blocks_kernel give every mask
// row to one wavefront: scores against all key-block means, softmax, and the cumulative-mass cut
// found without sorting, by bisection over the bit patterns of the (positive) probabilities.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "rapid_internal.h"
#include "rapid_mask.h"

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int MAX_NB = 2048;      // mask blocks per side the selection kernel holds in LDS

// Q and K of the joint sequence as one or two token segments (the image and the text stream of
// an MM-DiT block): token t < n0 is row t of segment 0, any other token row t - n0 of segment 1.
// Strides in elements, D contiguous; head and token strides are common to both segments.
struct QKView {
    const uint16_t* q0; const uint16_t* k0;
    const uint16_t* q1; const uint16_t* k1;      // null when there is one segment
    long long sb0, sb1, sh, sn;
    int n0, N, H;
    int kv_len;                                   // valid tokens of every sample, or
    const int32_t* kv_lens;                       // per sample (device, [B]), clamped to 0..N
    int text_start;
};

__device__ __forceinline__ int valid_tokens(const QKView& v, int b)
{
    if (v.kv_lens == nullptr) return v.kv_len;
    const int n = v.kv_lens[b];
    return n < 0 ? 0 : (n > v.N ? v.N : n);
}
// live blocks (those that start below the valid length) and the first text block of a sample
__device__ __forceinline__ void sample_blocks(const QKView& v, int b, int block, int nb, int& live, int& first_text)
{
    const int kv = valid_tokens(v, b);
    live = (kv + block - 1) / block;
    first_text = v.text_start < kv ? v.text_start / block : nb;
}

// means[(which, bh, i), :] = mean over the valid rows of block i of Q (which = 0) or K (1).  256 threads: D/8 column
// groups of 8 elements x 256/(D/8) row groups; every thread adds up its rows in increasing order, the row groups are
// then added in increasing order.  Bound by HBM: all loads of a block are requested before the first is used (one after the
// other where a last block is cut, a call of D = 128, 128-token blocks, N = 4221 took 15.4 us in place of 14.4), and
// STREAMED ones are non-temporal (H = 24, N = 16896, D = 128, 208 MB: 39.0 us in a loop, 36.8 requested at once, 33.1 =
// 6.3 TB/s non-temporal; N = 4608 13.9 / 13.0 / 11.0).  Only where Q and K are more than the caches keep for the attention
// that reads them next: at N = 4608 (57 MB) selection and attention in one call take 123.2 us, 124.1 when streamed.
template <int D, int BLOCK, bool STREAMED>
__global__ __launch_bounds__(256) void block_mean_kernel(const QKView v, int nb, float* __restrict__ means, size_t which_stride)
{
    constexpr int CG = D / 8, RG = 256 / CG, RPT = BLOCK / RG;
    __shared__ float red[RG][D];
    const int i = blockIdx.x % nb, bh = blockIdx.x / nb, which = blockIdx.y;
    const int b = bh / v.H, h = bh % v.H;
    const int lo = i * BLOCK;
    // (two segments: the first ends at a multiple of 128 tokens, so a block lies in one of them)
    const uint16_t* src = lo < v.n0 ? (which ? v.k0 : v.q0) + (size_t)b * v.sb0 : (which ? v.k1 : v.q1) + (size_t)b * v.sb1 - (size_t)v.n0 * v.sn;
    const int kv = valid_tokens(v, b);
    int hi = lo + BLOCK;
    hi = hi < kv ? hi : kv;                        // kv <= N: a ragged last block ends at N
    const int c = threadIdx.x % CG, g = threadIdx.x / CG;
    src += (size_t)h * v.sh + c * 8;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    auto add = [&](u32x4 x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc[2 * e] += __uint_as_float(x[e] << 16);
            acc[2 * e + 1] += __uint_as_float(x[e] & 0xffff0000u);
        }
    };
    if (lo < hi) {                                 // (rows past the last valid one: that one again, not added)
        u32x4 x[RPT];
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int r = lo + g + u * RG;
            const u32x4* at = (const u32x4*)(src + (size_t)(r < hi ? r : hi - 1) * v.sn);
            x[u] = STREAMED ? __builtin_nontemporal_load(at) : *at;
        }
#pragma unroll
        for (int u = 0; u < RPT; ++u)
            if (lo + g + u * RG < hi) add(x[u]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[g][c * 8 + e] = acc[e];
    __syncthreads();
    if (threadIdx.x < D) {
        float s = 0.f;
#pragma unroll
        for (int gg = 0; gg < RG; ++gg) s += red[gg][threadIdx.x];
        const int cnt = hi - lo;
        means[which * which_stride + ((size_t)bh * nb + i) * D + threadIdx.x] = cnt > 0 ? s / (float)cnt : 0.f;
    }
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
}
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// One wavefront per mask row (b, h, i); four rows per workgroup.
// What a row's result is written as: a byte per key-block into `mask` (when given), and/or the
// ascending list of kept key-blocks with its length (the form the attention kernels walk: the
// arrays `counts` and `index` of the attention workspace), so that selection can feed the
// attention without a byte mask in between.
struct RowSink {
    unsigned char* mask;     // [rows, nb] or null
    int32_t* counts;         // [rows] or null
    int32_t* index;          // [rows, nb], with counts
};

// One wavefront writes row `row`: keep(j) for j = lane, lane + 64, ...; every lane takes part.
template <class Keep>
__device__ __forceinline__ void write_row(const RowSink& sink, size_t row, int nb, int lane, Keep keep)
{
    int base = 0;
    for (int j0 = 0; j0 < nb; j0 += 64) {
        const int j = j0 + lane;
        const bool kp = j < nb && keep(j);
        if (sink.mask != nullptr && j < nb) sink.mask[row * nb + j] = kp ? 1 : 0;
        if (sink.counts != nullptr) {
            const unsigned long long bal = __ballot(kp);
            if (kp) sink.index[row * nb + base + __popcll(bal & ((1ull << lane) - 1ull))] = j;
            base += __popcll(bal);
        }
    }
    if (sink.counts != nullptr && lane == 0) sink.counts[row] = base;
}

template <int D>
__global__ __launch_bounds__(256) void select_blocks_kernel(const float* __restrict__ qmean, const float* __restrict__ kmean,
                                                            const QKView v, int block, int rows, int nb, float tau,
                                                            float scale, const RowSink sink)
{
    __shared__ float qrow[4][D];
    __shared__ float prob[4][MAX_NB];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wv;
    if (row >= rows) return;
    const int i = row % nb;
    const size_t bh = row / nb;
    int live, first_text;
    sample_blocks(v, (int)(bh / v.H), block, nb, live, first_text);
    if (i >= live) {
        write_row(sink, (size_t)row, nb, lane, [](int) { return false; });
        return;
    }
    for (int d = lane; d < D; d += 64) qrow[wv][d] = qmean[(size_t)row * D + d];
    __builtin_amdgcn_wave_barrier();               // one wavefront: its LDS accesses execute in order

    // scores of the live key-blocks (lane j, j + 64, ...), their maximum
    const float* kb = kmean + bh * nb * D;
    float mx = -INFINITY;
    for (int j = lane; j < live; j += 64) {
        const f32x4* kr = (const f32x4*)(kb + (size_t)j * D);
        float dot = 0.f;
#pragma unroll 4
        for (int d4 = 0; d4 < D / 4; ++d4) {
            const f32x4 kv = kr[d4];
            dot += qrow[wv][4 * d4] * kv[0];
            dot += qrow[wv][4 * d4 + 1] * kv[1];
            dot += qrow[wv][4 * d4 + 2] * kv[2];
            dot += qrow[wv][4 * d4 + 3] * kv[3];
        }
        const float s = scale * dot;
        prob[wv][j] = s;
        mx = fmaxf(mx, s);
    }
    mx = wave_max(mx);
    // unnormalised probabilities e = exp(s - max) <= 1 and their sum (normalising both sides
    // of "mass >= tau * total" changes nothing)
    float part = 0.f;
    for (int j = lane; j < live; j += 64) {
        const float e = expf(prob[wv][j] - mx);
        prob[wv][j] = e;
        part += e;
    }
    const float total = wave_sum(part);
    // v* = largest probability whose upper set {e >= v*} holds at least tau * total: positive
    // floats order like their bit patterns, and the mass of the upper set falls as the cut
    // rises, so bisect over the patterns between 0 and 1.0f.
    unsigned cut = 0u;
    if (tau < 1.0f) {
        const float target = tau * total;
        unsigned lo = 0u, hi = 0x3F800001u;                  // mass(lo) >= target > mass(hi) = 0
        while (hi - lo > 1u) {
            const unsigned mid = lo + (hi - lo) / 2u;
            float m = 0.f;
            for (int j = lane; j < live; j += 64) {
                const float e = prob[wv][j];
                m += (__float_as_uint(e) >= mid) ? e : 0.f;
            }
            m = wave_sum(m);
            if (m >= target) lo = mid; else hi = mid;
        }
        cut = lo;
    }
    const bool text_row = i >= first_text;
    write_row(sink, (size_t)row, nb, lane, [&](int j) {
        return j < live && (text_row || j >= first_text || j == i || __float_as_uint(prob[wv][j]) >= cut);
    });
}

// The same for up to SMALL_NB mask blocks per side (every shape of the paper's models): ROWS wavefronts take ROWS rows of one
// (sample, head).  Scores by fp32 MFMAs, tiles of 16 key-blocks dealt out to the wavefronts straight from the means in memory
// (a lane's 16 bytes of a row serve four MFMAs: the contraction index is a dummy); then a row per wavefront, its scores in
// registers.
// The cut: up to 64 blocks, block j is kept iff the blocks with a strictly larger probability hold less than tau of
// the mass, a sum each lane forms over all the others; beyond, the bisection of select_blocks_kernel between the smallest and
// the largest probability, which ends as soon as one value is left between the bounds (a dozen rounds of the thirty for scores
// that are spread out; from 0 on, near-equal scores, whose probabilities differ in their last bits only, took more).
// The kernel alone, us, H = 24, 132 blocks, D = 128: scores by vector instructions from LDS and the first cut 22.2; by MFMAs,
// bisection from 0 11.3, near-equal scores 11.9; from the smallest 10.5 and 10.0.
// ROWS = 16 reads the means of the keys half as often.  ROWS = 8 where its workgroups are still at most one per CU: half as many
// wavefronts share the vector unit of a CU, which counts once rows are long.  8 / 16 rows (and 4, no better), D = 128, (sample,
// head) pairs x blocks: 2 x 33 4.6 / 5.3 (4.8), 65 7.2 / 7.5 (7.5), 128 8.9 / 9.6 (8.4), 256 11.0 / 14.1 (10.4); 8 x 129 9.6 /
// 10.7 (10.9), 256 (128 workgroups of 16 rows) 10.8 / 13.8 (14.9); 24 x 48 5.0 / 5.4 (5.8), 65 7.7 / 8.1 (8.9).
constexpr int SMALL_NB = 256;

// v of all 64 lanes combined, the same in all of them: shifts inside rows of 16 lanes, then the last lane of rows 0 and 2
// to rows 1 and 3, then lane 31 to rows 2 and 3; a lane without a source takes `none`.  All lanes active.
template <class Op>
__device__ __forceinline__ float wave_combine(float v, float none, Op op)
{
    auto moved = [&](auto ctrl, auto rows) {
        return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(none), __float_as_int(v), decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
    };
    typedef std::integral_constant<int, 0xf> all;
    v = op(v, moved(std::integral_constant<int, 0x111>(), all()));
    v = op(v, moved(std::integral_constant<int, 0x112>(), all()));
    v = op(v, moved(std::integral_constant<int, 0x114>(), all()));
    v = op(v, moved(std::integral_constant<int, 0x118>(), all()));
    v = op(v, moved(std::integral_constant<int, 0x142>(), std::integral_constant<int, 0xa>()));
    v = op(v, moved(std::integral_constant<int, 0x143>(), std::integral_constant<int, 0xc>()));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_total(float v) { return wave_combine(v, 0.f, [](float a, float b) { return a + b; }); }

template <int D, int U, int ROWS>              // U: 64-block stretches of a row; ROWS: per workgroup
__global__ __launch_bounds__(64 * ROWS, 4) void select_blocks_small_kernel(const float* __restrict__ qmean,
                                                                   const float* __restrict__ kmean, const QKView v,
                                                                   int block, int nb, float tau, float scale,
                                                                   const RowSink sink)
{
    constexpr int ROW = 64 * U + 4;
    __shared__ __attribute__((aligned(16))) float ps[ROWS][ROW];
    const int groups = (nb + ROWS - 1) / ROWS;
    const size_t bh = blockIdx.x / groups;
    int live, first_text;
    sample_blocks(v, (int)(bh / v.H), block, nb, live, first_text);
    const int i0 = (blockIdx.x % groups) * ROWS;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    for (int k0 = wv * 16; k0 < live; k0 += ROWS * 16) {
        const int kr = k0 + n, qr = i0 + n % ROWS; // (columns from ROWS on of the product: the rows again, not stored)
        const f32x4* kp = (const f32x4*)(kmean + (bh * nb + (kr < live ? kr : live - 1)) * D) + g;
        const f32x4* qp = (const f32x4*)(qmean + (bh * nb + (qr < live ? qr : live - 1)) * D) + g;
        f32x4 kf[D / 16], qf[D / 16];
#pragma unroll
        for (int t = 0; t < D / 16; ++t) { kf[t] = kp[4 * t]; qf[t] = qp[4 * t]; }
#pragma unroll
        for (int t = 0; t < D / 16; ++t) asm volatile("" : "+v"(kf[t]), "+v"(qf[t]));    // all on their way at once
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < D / 16; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][e], qf[t][e], acc, 0, 0, 0);
        f32x4 out;
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] = scale * acc[r];
        if (n < ROWS) *(f32x4*)(&ps[n][k0 + 4 * g]) = out;      // key-blocks 4 g .. of the tile, query row n
    }
    __syncthreads();

    const int i = i0 + wv;
    if (i >= nb) return;
    const size_t mrow = bh * nb + i;
    if (i >= live) {
        write_row(sink, mrow, nb, lane, [](int) { return false; });
        return;
    }
    float e[U], mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        e[u] = lane + 64 * u < live ? ps[wv][lane + 64 * u] : -INFINITY;
        mx = fmaxf(mx, e[u]);
    }
    mx = wave_combine(mx, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
    float part = 0.f, least = INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool in = lane + 64 * u < live;
        e[u] = in ? expf(e[u] - mx) : 0.f;
        least = in ? fminf(least, e[u]) : least;
        part += e[u];
    }
    const float target = tau * wave_total(part);
    const bool text_row = i >= first_text;
    bool kept[U];
    if constexpr (U == 1) {
        ps[wv][lane] = e[0];                       // (a wavefront's own row; zeros past the live blocks)
        __builtin_amdgcn_wave_barrier();
        float above = 0.f;                         // mass of the blocks that come before this one
        for (int j = 0; j < live; j += 4) {
            const f32x4 x = *(const f32x4*)(&ps[wv][j]);
#pragma unroll
            for (int r = 0; r < 4; ++r) above += x[r] > e[0] ? x[r] : 0.f;
        }
        kept[0] = above < target;
    } else {
        unsigned lo = __float_as_uint(wave_combine(least, INFINITY, [](float a, float b) { return fminf(a, b); }));
        unsigned hi = 0x3F800001u;                 // mass(lo) >= target > mass(hi) = 0
        int from_lo = 64 * U, from_hi = 0;         // values at or above either, at most
        if (!(target > 0.f)) lo = hi = ~0u;        // not a number: only what is kept in any case
        while (hi - lo > 1u && from_lo - from_hi > 1) {
            const unsigned mid = lo + (hi - lo) / 2u;
            float m = 0.f;
            int from_mid = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = __float_as_uint(e[u]) >= mid;
                m += in ? e[u] : 0.f;
                from_mid += __popcll(__builtin_amdgcn_ballot_w64(in));
            }
            const bool enough = wave_total(m) >= target;
            if (enough) { lo = mid; from_lo = from_mid; }
            else { hi = mid; from_hi = from_mid; }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) kept[u] = __float_as_uint(e[u]) >= lo;
    }
    write_row(sink, mrow, nb, lane, [&](int j) {
        if (j >= live) return false;
        bool k = false;
#pragma unroll
        for (int u = 0; u < U; ++u) k = j / 64 == u ? kept[u] : k;
        return k || text_row || j >= first_text || j == i || tau >= 1.0f;
    });
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

size_t means_bytes(int B, int H, int nb, int D) { return (size_t)2 * B * H * nb * D * sizeof(float); }

bool shape_ok(int B, int H, int N, int D, int block, bool ragged)
{
    if (B <= 0 || H <= 0 || N <= 0 || N > (1 << 22)) return false;
    if ((long long)B * H > 0x7fffffffLL / 4096) return false;
    if (D != 64 && D != 128) return false;
    if (block != 64 && block != 128) return false;
    if (!ragged && N % block != 0) return false;
    if ((N + block - 1) / block > MAX_NB) return false;
    return true;
}

// One validated call: means, then the selection kernel that fits the size.
int run_select(const QKView& v, int B, int D, int block, float tau, float scale, const RowSink& sink, void* workspace,
               size_t workspace_bytes, void* stream)
{
    const int H = v.H, nb = (v.N + block - 1) / block;
    if (nb > MAX_NB) return RAPID_ERR_UNSUPPORTED;
    const size_t need = means_bytes(B, H, nb, D);
    if (!workspace || workspace_bytes < need) return RAPID_ERR_WORKSPACE;
    if (!aligned16(workspace)) return RAPID_ERR_ALIGN;
    if ((long long)B * H * nb > 0x7fffffffLL / 16) return RAPID_ERR_SHAPE;
    if (!(scale > 0.f)) scale = 1.0f / sqrtf((float)D);

    float* means = (float*)workspace;
    const size_t which_stride = (size_t)B * H * nb * D;
    hipStream_t s = (hipStream_t)stream;
    const dim3 g1((unsigned)(nb * B * H), 2u);
    // Half of the 256 MB memory-side cache.  us, plain loads / streamed, selection alone right after Q and K were written, H = 24,
    // D = 128, MB of Q and K: 28 13.2 14.0; 57 17.5 17.9; 88 22.6 22.6; 126 30.6 30.3; 151 34.4 34.6; 208 49.6 46.0; 415 118.5
    // 90.9 (the same tensors again and again, 208: 43.4 47.0; others in turn: 49.5 46.7).  Selection and attention in one call:
    // 28 67.3 69.8; 57 124.5 125.9; 126 to 415 the same within 1 %.
    const bool streamed = 4.0 * B * H * v.N * D > 128e6;
    const auto pick_mean = [&](auto d, auto bl) {
        constexpr int DD = decltype(d)::value, BB = decltype(bl)::value;
        return streamed ? block_mean_kernel<DD, BB, true> : block_mean_kernel<DD, BB, false>;
    };
    typedef std::integral_constant<int, 64> c64;
    typedef std::integral_constant<int, 128> c128;
    const auto mean = D == 64 ? (block == 64 ? pick_mean(c64(), c64()) : pick_mean(c64(), c128()))
                              : (block == 64 ? pick_mean(c128(), c64()) : pick_mean(c128(), c128()));
    hipLaunchKernelGGL(mean, g1, dim3(256), 0, s, v, nb, means, which_stride);
    if (hipGetLastError() != hipSuccess) return RAPID_ERR_DEVICE;

    const int rows = B * H * nb;
    if (nb <= SMALL_NB) {
        typedef std::integral_constant<int, 8> c8;
        typedef std::integral_constant<int, 16> c16;
        const int per = nb > 32 && (long long)B * H * ((nb + 15) / 16) <= 128 ? 8 : 16;
        const dim3 gs((unsigned)(B * H * ((nb + per - 1) / per)));
        const auto pick = [&](auto d, auto r) {
            constexpr int DD = decltype(d)::value, RR = decltype(r)::value;
            return nb <= 64 ? select_blocks_small_kernel<DD, 1, RR> : nb <= 128 ? select_blocks_small_kernel<DD, 2, RR>
                 : nb <= 192 ? select_blocks_small_kernel<DD, 3, RR> : select_blocks_small_kernel<DD, 4, RR>;
        };
        const auto select = D == 64 ? (per == 8 ? pick(c64(), c8()) : pick(c64(), c16()))
                                    : (per == 8 ? pick(c128(), c8()) : pick(c128(), c16()));
        hipLaunchKernelGGL(select, gs, dim3(64 * per), 0, s, means, means + which_stride, v, block, nb, tau, scale, sink);
        return hipGetLastError() == hipSuccess ? RAPID_OK : RAPID_ERR_DEVICE;
    }
    const dim3 g2((unsigned)((rows + 3) / 4));
    if (D == 64)
        hipLaunchKernelGGL((select_blocks_kernel<64>), g2, dim3(256), 0, s, means, means + which_stride, v, block, rows, nb,
                           tau, scale, sink);
    else
        hipLaunchKernelGGL((select_blocks_kernel<128>), g2, dim3(256), 0, s, means, means + which_stride, v, block, rows, nb,
                           tau, scale, sink);
    return hipGetLastError() == hipSuccess ? RAPID_OK : RAPID_ERR_DEVICE;
}

// Q and K of the joint sequence from segment descriptors, validated (v and o are not looked at).
int joint_view(const rapid_attn_segment* segments, int n_segments, int B, int H, int D, int block, int kv_len,
               const int* kv_lens, int text_start, float tau, QKView& v)
{
    if (!segments) return RAPID_ERR_NULL;
    if (n_segments != 1 && n_segments != 2) return RAPID_ERR_SHAPE;
    if (B <= 0 || H <= 0) return RAPID_ERR_SHAPE;
    if ((long long)B * H > 0x7fffffffLL / 4096) return RAPID_ERR_SHAPE;
    if (D != 64 && D != 128) return RAPID_ERR_UNSUPPORTED;
    if (block != 64 && block != 128) return RAPID_ERR_UNSUPPORTED;
    if (text_start < 0 || !(tau > 0.f)) return RAPID_ERR_SHAPE;
    long long N = 0;
    rapid_attn_segment seg[2];                    // strides of size-1 dimensions are not looked at
    for (int i = 0; i < n_segments; ++i) seg[i] = rapid_internal::normalised_segment(segments[i], B, H, i == 1 ? &seg[0] : nullptr);
    segments = seg;
    for (int i = 0; i < n_segments; ++i) {
        const rapid_attn_segment& g = segments[i];
        if (!g.q || !g.k) return RAPID_ERR_NULL;
        if (g.n <= 0) return RAPID_ERR_SHAPE;
        if (!aligned16(g.q) || !aligned16(g.k)) return RAPID_ERR_ALIGN;
        const long long st[3] = {g.in_stride_b, g.in_stride_h, g.in_stride_n};
        for (int j = 0; j < 3; ++j) {
            if (st[j] < 0 || st[j] > (1LL << 40)) return RAPID_ERR_SHAPE;
            if (st[j] % 8 != 0) return RAPID_ERR_ALIGN;        // every row starts on 16 bytes
        }
        if (g.in_stride_n < D || g.in_stride_n > (1LL << 23)) return RAPID_ERR_SHAPE;
        N += g.n;
    }
    if (N > (1 << 22)) return RAPID_ERR_SHAPE;
    if (n_segments == 2) {
        // as rapid_attn_joint: the masks made here are for that call
        if (segments[0].n % 128 != 0) return RAPID_ERR_SHAPE;
        if (segments[0].in_stride_h != segments[1].in_stride_h || segments[0].in_stride_n != segments[1].in_stride_n)
            return RAPID_ERR_SHAPE;
    }
    if (kv_len == 0) kv_len = (int)N;
    if (kv_len < 1 || kv_len > N) return RAPID_ERR_SHAPE;
    v.q0 = (const uint16_t*)segments[0].q; v.k0 = (const uint16_t*)segments[0].k;
    v.q1 = n_segments == 2 ? (const uint16_t*)segments[1].q : nullptr;
    v.k1 = n_segments == 2 ? (const uint16_t*)segments[1].k : nullptr;
    v.sb0 = segments[0].in_stride_b; v.sb1 = n_segments == 2 ? segments[1].in_stride_b : 0;
    v.sh = segments[0].in_stride_h; v.sn = segments[0].in_stride_n;
    v.n0 = n_segments == 2 ? segments[0].n : (int)N; v.N = (int)N; v.H = H;
    v.kv_len = kv_len; v.kv_lens = kv_lens; v.text_start = text_start;
    return RAPID_OK;
}

}  // namespace

namespace rapid_internal {

size_t select_scratch_bytes(int B, int H, int nb, int D) { return means_bytes(B, H, nb, D); }

int select_to_lists(const rapid_attn_segment* segments, int n_segments, int B, int H, int D, int block,
                    int kv_len, const int* kv_lens, int text_start, float tau, float scale,
                    unsigned char* mask, int32_t* counts, int32_t* index, void* scratch, size_t scratch_bytes,
                    void* stream)
{
    if (!counts || !index) return RAPID_ERR_NULL;
    QKView v{};
    const int rc = joint_view(segments, n_segments, B, H, D, block, kv_len, kv_lens, text_start, tau, v);
    if (rc != RAPID_OK) return rc;
    return run_select(v, B, D, block, tau, scale, RowSink{mask, counts, index}, scratch, scratch_bytes, stream);
}

}  // namespace rapid_internal

extern "C" {

int rapid_mask_select(const void* q, const void* k, int B, int H, int N, int D, int block, int kv_len,
                      int text_start, float tau, float scale, unsigned char* mask, void* workspace,
                      size_t workspace_bytes, void* stream)
{
    if (!q || !k || !mask) return RAPID_ERR_NULL;
    if (B <= 0 || H <= 0 || N <= 0 || N > (1 << 22)) return RAPID_ERR_SHAPE;
    if ((long long)B * H > 0x7fffffffLL / 4096) return RAPID_ERR_SHAPE;
    if (kv_len < 1 || kv_len > N || text_start < 0 || !(tau > 0.f)) return RAPID_ERR_SHAPE;
    if (D != 64 && D != 128) return RAPID_ERR_UNSUPPORTED;
    if (block != 64 && block != 128) return RAPID_ERR_UNSUPPORTED;
    if (N % block != 0) return RAPID_ERR_SHAPE;
    if (N / block > MAX_NB) return RAPID_ERR_UNSUPPORTED;
    if (!aligned16(q) || !aligned16(k)) return RAPID_ERR_ALIGN;
    QKView v{};
    v.q0 = (const uint16_t*)q; v.k0 = (const uint16_t*)k; v.q1 = nullptr; v.k1 = nullptr;
    v.sb0 = (long long)H * N * D; v.sb1 = 0; v.sh = (long long)N * D; v.sn = D;
    v.n0 = N; v.N = N; v.H = H;
    v.kv_len = kv_len; v.kv_lens = nullptr; v.text_start = text_start;
    return run_select(v, B, D, block, tau, scale, RowSink{mask, nullptr, nullptr}, workspace, workspace_bytes, stream);
}

int rapid_mask_select_joint(const rapid_attn_segment* segments, int n_segments, int B, int H, int D, int block,
                            int kv_len, const int* kv_lens, int text_start, float tau, float scale,
                            unsigned char* mask, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!mask) return RAPID_ERR_NULL;
    QKView v{};
    const int rc = joint_view(segments, n_segments, B, H, D, block, kv_len, kv_lens, text_start, tau, v);
    if (rc != RAPID_OK) return rc;
    return run_select(v, B, D, block, tau, scale, RowSink{mask, nullptr, nullptr}, workspace, workspace_bytes, stream);
}

size_t rapid_mask_select_workspace_bytes(int B, int H, int N, int D, int block)
{
    if (!shape_ok(B, H, N, D, block, false)) return 0;
    return means_bytes(B, H, N / block, D);
}

size_t rapid_mask_select_joint_workspace_bytes(int B, int H, int N, int D, int block)
{
    if (!shape_ok(B, H, N, D, block, true)) return 0;
    return means_bytes(B, H, (N + block - 1) / block, D);
}

float rapid_mask_level_tau(int action)
{
    switch (action) {
        case 0: return 1.0f;
        case 1: return 0.98f;
        case 2: return 0.95f;
        case 3: return 0.90f;
        default: return NAN;
    }
}

}  // extern "C"
