// MM-DiT joint attention for MI355X (gfx950): dense and block-sparse, flash-style.
//
// Operation: RAPID^3 Sec. 3.1 Eq. 1 (self-attention block of a DiT layer) and
// Sec. 3.2 Level-3 / Eq. 4 (the same block restricted to a pruned attention map,
// per layer and per head).  The pruned map is given as a block mask; pruned tiles
// are never read.
//
// Building blocks of attn_sparse_sg_kernel<64> (a wavefront owns 32 queries and walks over 64-key tiles; the others
// are described at the stream):
//   S^T = K Q^T    v_mfma_f32_32x32x16_bf16, A = K tile rows from LDS (128-bit
//                  reads), B = the wavefront's Q rows held in registers for the
//                  whole kernel.  Computing the TRANSPOSED score tile puts one
//                  query per lane: the running max / sum are per-lane scalars, the
//                  row reductions are in-register plus ONE cross-half exchange
//                  (v_permlane32_swap), and the fp32 accumulator registers of a
//                  lane are, after conversion to bf16, exactly the B operand of
//                  the next product -- P never touches LDS.
//   O^T += V^T P^T same MFMA; A = V^T fragments fetched straight out of the
//                  row-major V tile with the LDS transpose read
//                  (ds_read_b64_tr_b16), B = P^T from the registers above.
//                  The contraction index is a dummy, so the key order inside a
//                  16-key step is whatever the accumulator layout yields (keys
//                  4h+r and 8+4h+r for lane half h); V^T is fetched in that order.
//   tiles          global -> LDS directly (global_load_lds_dwordx4), chunk-swizzled,
//                  several tiles ahead of their use.
// Kernels:
//   attn_dense_stream_kernel<D> dense: 256 queries per workgroup (the last, partly filled round of an XCD
//                               in halves, quarters or pieces of 192), on the 16x16x32 stream described there
//   attn_dense_pp_kernel<D>     dense, small problems: 32 queries per workgroup, the keys split between
//                               two groups of wavefronts
//   attn_sparse_sg_kernel<D>    sparse, 128-token mask tiles: one four-wavefront workgroup per plan
//                               record (a query-block or a piece of its kept list); pieces are
//                               merged by the last one to finish.  D = 128 on the 16x16x32 stream
//   attn_sparse_wide_kernel     the same at D = 64 on the stream, for calls of many rows
//   attn_sparse_pp_kernel<D>    sparse, 64-token mask tiles: one query-block per workgroup on the stream, the
//                               keys of a block split between two groups of wavefronts
//   plan_small_kernel           launch plan in one launch, from the mask or from counts (up to 64 blocks per side); the
//                               attention kernels then read their rows of the mask themselves, and where all rows
//                               are on the chip at once they need no plan either
//   compact_mask_kernel, plan_split_kernel (128-token tiles), plan_kernel (64-token tiles)
//                               lists and plan in two launches for larger problems
// Entry points (C ABI, bottom of the file): rapid_attn_dense, rapid_attn_block_sparse,
// rapid_attn_block_sparse_static (scratch in a fixed array of this file), rapid_attn_joint,
// rapid_attn_joint_select (selection kernels of rapid_mask.hip write the kept lists).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <initializer_list>
#include <type_traits>

#include "rapid_attn.h"
#include "rapid_internal.h"
#include "rapid_mask.h"

// Scratch of the entry point that allocates nothing (see static_scratch below).
static __device__ __align__(256) unsigned char scratch[RAPID_ATTN_STATIC_SCRATCH_BYTES];

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int KT = 64;          // keys per LDS tile
constexpr int XCDS = 8;         // L2 domains the dispatcher deals workgroups over
constexpr int DENSE_QT = 256;    // query rows per workgroup on the dense path
constexpr float LOG2E = 1.44269504088896340736f;

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

// A [B, H, tokens, D] tensor handed over as one or two token segments: token t < n0 is row t
// of segment 0, any other token row t - n0 of segment 1 (MM-DiT keeps the image and the
// text stream in separate tensors and joins them only for attention).  Strides in elements,
// D contiguous; head and token strides are common to both segments, all strides to Q, K and V.
struct SegTensor {
    const __bf16* seg0;
    const __bf16* seg1;      // of no use when there is one segment
};
struct SegStrides {
    long long sb0, sb1;      // batch strides
    long long sh, sn;        // head stride, token stride
};

// The token rows of one (sample, head): row r starts at (r < n0 ? base0 : base1) + r * row_bytes
// (base1 is biased by -n0 rows so that both segments are indexed by the joint token number).
struct Rows {
    const char* base0;
    const char* base1;
    int n0;
    unsigned row_bytes;
    __device__ __forceinline__ const char* row(int r) const { return (r < n0 ? base0 : base1) + (size_t)r * row_bytes; }
};

__device__ __forceinline__ Rows rows_of(const SegTensor& t, const SegStrides& s, int b, int h, int n0)
{
    const long long head = h * s.sh;
    Rows r;
    r.base0 = (const char*)(t.seg0 + (b * s.sb0 + head));
    r.base1 = (const char*)(t.seg1 + (b * s.sb1 + head - n0 * s.sn));
    r.n0 = n0;
    r.row_bytes = (unsigned)(s.sn * 2);
    return r;
}

// A divisor that only the host knows.  n / d in scalar code is a division by way of vector floats, 35 instructions; as a high
// product with magic = ceil(2^32 / d) it is exact while n * d < 2^32 (what it is too large by is less than n * d / 2^32 / d).
// magic = 0: by division (d = 1, or dividends that large).
struct Divisor {
    int d;
    unsigned magic;
    __device__ __forceinline__ int of(int n) const
    {
        if (magic != 0u) return (int)__umulhi((unsigned)n, magic);
        return d == 1 ? n : __builtin_amdgcn_readfirstlane(n / d);
    }
};
inline Divisor divisor(int d, long long dividends)
{
    return {d, d > 1 && dividends * d < 0x100000000LL ? 0xffffffffu / (unsigned)d + 1u : 0u};
}

struct AttnParams {
    SegTensor q, k, v, o;
    SegStrides in, out;      // of Q, K and V; of O
    const int32_t* kv_lens;  // per-sample valid tokens (device, [B]) or null: kv_len for all
    int n0;                  // tokens in the first segment (N when there is one)
    const unsigned char* mask;    // sparse: the block mask where the kernels read their rows of it themselves, else null
    int32_t* counts;         // sparse: kept key-blocks per (b,h,query-block); dense: null
    int32_t* order;          // sparse: launch plan (64-token tiles: item ids; 128-token tiles: PlanRec records)
    int32_t* index;          // sparse: kept key-block lists, nb per row
    int32_t* arrived;        // sparse, 128-token tiles: finished pieces per split item
    char* partial;           // sparse, 128-token tiles: partial results of the pieces of split items
    int N, kv_len;
    Divisor H;
    int turn;                // dense: see dense_run
    int pairs;               // sparse: (sample, head) pairs (here, where it comes with what rows are looked up by; alone it is a load more)
    Divisor nq;              // query tiles per (sample, head)
    int items;               // B*H*nq
    int chunk;               // ceil(items / XCDS)
    int whole, cut;          // dense: whole items of an XCD, pieces of each of the others (3: pieces of 192 queries)
    int nb;                  // mask blocks per side (sparse only)
    int segs;                // sparse: plan segments that hold items, min(XCDS, B*H)
    unsigned seg_magic;      // ceil(2^32 / segs)
    int planned;             // sparse: PLAN_NONE, PLAN_FOUND or PLAN_READ
    int pmax;                // sparse, 128-token tiles: partial-result slots per segment
    float c;                 // scale * log2(e)
};

// Where a workgroup of the sparse path has its row from (see sparse_work): its number; what every workgroup finds out about all rows
// of its segment; the plan in `order`.
enum { PLAN_NONE, PLAN_FOUND, PLAN_READ };

// All arguments on their way with the first of them: what the compiler loads where it is needed, one behind the other, is a trip
// to memory each time.  us, without / with, 128-token masks, D = 64: H = 8, N = 8192, 0.2 130.6 / 126.3; H = 24, N = 2048, 0.3
// 31.3 / 30.8, 1024 14.6 / 14.3; the kernels of the stream, which loaded them early anyway, the same.
__device__ __forceinline__ void arguments_at_hand(const AttnParams& p)
{
    asm volatile("" ::"s"(p.q.seg0), "s"(p.k.seg0), "s"(p.v.seg0), "s"(p.o.seg0), "s"(p.in.sb0), "s"(p.in.sh), "s"(p.out.sb0), "s"(p.out.sn),
                 "s"(p.kv_lens), "s"(p.mask), "s"(p.index), "s"(p.partial), "s"(p.H.magic), "s"(p.chunk), "s"(p.c));
}

// Valid tokens of a sample: clamped to 0..N where they are given per sample.
__device__ __forceinline__ int valid_tokens(const AttnParams& p, int smp)
{
    int kv_len = p.kv_len;
    if (p.kv_lens != nullptr) {
        kv_len = ((const __attribute__((address_space(4))) int32_t*)p.kv_lens)[smp];
        kv_len = kv_len < 0 ? 0 : (kv_len > p.N ? p.N : kv_len);
        kv_len = __builtin_amdgcn_readfirstlane(kv_len);   // (the clamp is a vector instruction)
    }
    return kv_len;
}

// ---------------------------------------------------------------------------
// Mask compaction: one wavefront per (b, h, query-block) row of the mask.
// counts[row] = number of kept key-blocks whose first token is below kv_len;
// index[row*nb + 0..count) = those key-blocks, ascending.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void compact_mask_kernel(
    const unsigned char* __restrict__ mask, int rows, int nb, int block, int kv_len,
    const int32_t* __restrict__ kv_lens, int rows_per_sample, int N,
    int32_t* __restrict__ counts, int32_t* __restrict__ index)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    if (kv_lens != nullptr) {
        kv_len = kv_lens[row / rows_per_sample];
        kv_len = kv_len < 0 ? 0 : (kv_len > N ? N : kv_len);
    }
    const unsigned char* mrow = mask + (size_t)row * nb;
    int32_t* irow = index + (size_t)row * nb;
    int base = 0;
    for (int j0 = 0; j0 < nb; j0 += 64) {
        const int j = j0 + lane;
        const bool keep = (j < nb) && (mrow[j] != 0) && ((long long)j * block < kv_len);
        const unsigned long long bal = __ballot(keep);
        if (keep) irow[base + __popcll(bal & ((1ull << lane) - 1ull))] = j;
        base += __popcll(bal);
    }
    if (lane == 0) counts[row] = base;
}

// ---------------------------------------------------------------------------
// Launch plans of the sparse path.  Items = (b, h, query-block).  All items of one (b,h)
// go to XCD (b*H + h) % 8, so the K/V of a head stay in one L2; inside an XCD the entries
// are ordered by length, longest first (the dispatcher hands out workgroups in id order, so
// this is longest-processing-time-first scheduling of a ragged batch).  One workgroup per
// XCD: counting sort over the lengths.  Entries of equal length land in arbitrary order;
// that only changes which workgroup computes an entry, never its value.
// ---------------------------------------------------------------------------
constexpr int PLAN_MAX_NB = 8176;                // bins 0 .. nb fit the scan below
constexpr int PLAN_BINS = 8192;                  // 8 bins per thread

constexpr int PLAN_CACHE = 4096;                 // counts of this many items are kept in LDS

// Inclusive prefix sum over the 64 lanes of a wavefront with data-parallel-primitive moves:
// four shifts inside each row of 16 lanes, then lane 15 of rows 0 and 2 is added to rows 1
// and 3, then lane 31 to rows 2 and 3.  A lane without a source takes 0.  All lanes active.
__device__ __forceinline__ int wave_scan_inclusive(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return v;
}

// Maximum over the 64 lanes, valid in lane 63 (same moves; a lane without a source keeps its own).
__device__ __forceinline__ int wave_max_to_last(int v)
{
    auto step = [&](int t) { v = t > v ? t : v; };
    step(__builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
    return v;
}

// Exclusive prefix sum of one value per thread over the 1024 threads of the block: a scan
// inside each wavefront, then the 16 wavefront totals through LDS.  Two barriers.
__device__ __forceinline__ int plan_block_scan(int v, int* wave_sum, int tid)
{
    const int lane = tid & 63, wv = tid >> 6;
    const int incl = wave_scan_inclusive(v);
    if (lane == 63) wave_sum[wv] = incl;
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {                // all 16 reads in flight, none depends on wv
        const int t = wave_sum[w];
        before += w < wv ? t : 0;
    }
    __syncthreads();
    return before + incl - v;
}

// Exclusive prefix sum of hist[0 .. PLAN_BINS) in place (thread t owns bins 8t..8t+7).
__device__ __forceinline__ void plan_scan_bins(int* hist, int* wave_sum, int tid)
{
    int own[8], sum = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) { own[j] = hist[8 * tid + j]; sum += own[j]; }
    int run = plan_block_scan(sum, wave_sum, tid);
#pragma unroll
    for (int j = 0; j < 8; ++j) { hist[8 * tid + j] = run; run += own[j]; }
    __syncthreads();
}

// 64-token mask tiles: order[x * chunk + i] = i-th item of XCD x, -1 past the end.
__global__ __launch_bounds__(1024) void plan_kernel(const int32_t* __restrict__ counts, int BH, int nb, int chunk,
                                                    int32_t* __restrict__ order)
{
    __shared__ int hist[PLAN_BINS];              // by r = nb - count (r = 0: longest)
    __shared__ int wave_sum[16];
    const int x = blockIdx.x, tid = threadIdx.x;
    const int n_bh = (BH - x + XCDS - 1) / XCDS;  // (b,h) pairs with index % 8 == x
    const int n_items = n_bh > 0 ? n_bh * nb : 0;
    int32_t* out = order + (size_t)x * chunk;
    auto item_of = [&](int i) { return ((i / nb) * XCDS + x) * nb + i % nb; };
    if (nb > PLAN_MAX_NB) {                       // no sort: natural order
        for (int i = tid; i < chunk; i += 1024) out[i] = i < n_items ? item_of(i) : -1;
        return;
    }
    for (int i = tid; i < chunk; i += 1024) out[i] = -1;
#pragma unroll
    for (int j = 0; j < 8; ++j) hist[8 * tid + j] = 0;
    __syncthreads();
    for (int i = tid; i < n_items; i += 1024) atomicAdd(&hist[nb - counts[item_of(i)]], 1);
    __syncthreads();
    plan_scan_bins(hist, wave_sum, tid);
    for (int i = tid; i < n_items; i += 1024) {
        const int item = item_of(i);
        out[atomicAdd(&hist[nb - counts[item]], 1)] = item;
    }
}

// 128-token mask tiles: the plan is a list of records, one per workgroup.  The dispatcher
// fills the CUs entry by entry, so an entry that is long against a CU's share of the work
// leaves most of the chip idle at the end: an item can be cut into P pieces (SplitRule
// below).  Each piece is a record of its own; the pieces leave partial results in the
// workspace and the last one to finish combines them.  A piece is expensive (its partial
// result goes through memory: at D = 128 an entry costs about two key-blocks of
// time and a piece two more), so only rows several times the average (the text rows of a
// sparse mask) are worth cutting.  Partial-result slots are handed out in item order (a
// prefix sum, so the plan does not depend on timing); an item that no longer fits in the
// XCD's pmax slots stays whole.
struct PlanRec {
    int item;     // b*H*nb + h*nb + query-block, or -1: no work
    int blk0;     // first position of the piece in the item's kept list
    int nblk;     // kept key-blocks of the piece
    int w;        // -1: the whole item; else (first partial slot << 8) | (piece << 4) | (P - 1)
};
constexpr int CUS_PER_XCD = 32;                  // MI355X: 256 CUs in 8 XCDs
// Segments of the plan that the chip is dealt out to, and the CUs that work on one: an XCD's, or, with few (sample, head)
// pairs, its share of all of them (see entry_of).
constexpr __host__ __device__ int segments(int BH, int nb, int block)
{
    return nb >= 24 && BH < (block == 128 ? XCDS : XCDS / 2 + 1) ? BH : XCDS;
}
constexpr __host__ __device__ int segment_cus(int BH, int nb, int block) { return CUS_PER_XCD * XCDS / segments(BH, nb, block); }
constexpr int SPLIT_MIN_BLOCKS = 8;
constexpr int SPLIT_MAX_PIECES = 16;
constexpr int SPLIT_SLOTS = 256;                 // partial-result slots per segment, at most (and one per item: workspace_layout)
constexpr int ENTRY_COST = 2, PIECE_COST = 2;    // in key-blocks of time at D = 128
// (Taken from the loop of 32x32x16 MFMAs; on the stream, over 21 shapes by 6 densities at D = 128, costs of 1 and 1 are
// 0.1 % faster on all-ones masks in the mean (3.4 % at best), 3 and 3 0.4 % slower there (10.9 % at worst), and 2 or 3
// granules per CU in place of 2.5 within 0.3 % in the mean, -6 to +1 % case by case.)

// The rule of one XCD.  P(c) = round(c * g / total) pieces for an item with c kept key-blocks
// (g granules: pieces of about total / g), or p_all pieces for every item when that is set;
// in both cases at most c / SPLIT_MIN_BLOCKS and SPLIT_MAX_PIECES, at least 1.  A segment of more than 32 CUs: as many in
// place of 32, but no more granules than partial-result slots (or than 32 CUs get): they are handed out in item order, and the
// text rows, which need them most, come last (H = 2, N = 16896, density 0.1, D = 128: 282 us without that limit).  The slots of
// a segment are not more for having more CUs, so long rows that are nearly alike stay whole there and leave CUs idle.
//   D = 128: g = 32 CUs x 2.5.  Rows that are all about alike (the longest within 1/9 of the
//     mean: an all-ones mask) are not told apart by their lengths; what matters then is how
//     many rounds the 64 places of the XCD need, so p_all is the P that minimises
//     rounds(P) * (piece length + cost of an entry), the first such P.  There may be slots for the pieces of the first rows
//     only.  Where rows outnumber CUs that still fills the last round; with a CU for every row the call lasts as long as
//     the rows that stay whole, so then a P counts only if all of them get their slots.  us, H heads, all ones, some rows in pieces
//     / none: rows <= CUs 4, N = 6144 113.5 / 105.7; 5, 4608 88.5 / 82.2; 7, 4608 93.6 / 84.0; rows > CUs 2, 16896 298 / 341;
//     4, 16896 480 / 678; 6, 12288 402 / 496.
//   D = 64: g = 32 x 4; rows all alike: 32 x 12 (fewer items than the 128 places: cut them all).
struct SplitRule {
    int g;
    int p_all;     // 0: by length
};

// cost of cutting every one of n_items rows of max_c blocks into P pieces, D = 128 (T: wide enough for n_items * P * max_c)
template <class T>
__device__ __forceinline__ T split_alike_cost(int cus, int n_items, int max_c, int P)
{
    const T places = cus * 2;
    const T rounds = ((T)n_items * P + places - 1) / places;
    return rounds * ((max_c + P - 1) / P + ENTRY_COST + (P > 1 ? PIECE_COST : 0));
}

__device__ __forceinline__ bool rows_alike(int n_items, int max_c, unsigned long long total)
{
    return 8ull * (unsigned long long)n_items * (unsigned)max_c <= 9ull * total;
}

// `costs` holds split_alike_cost for P = 1 .. SPLIT_MAX_PIECES (used at D = 128 when the rows are alike)
template <class T>
__device__ __forceinline__ SplitRule split_rule(int D, int cus, int pmax, int n_items, int max_c, unsigned long long total, const T* costs)
{
    SplitRule r;
    r.p_all = 0;
    const bool alike = rows_alike(n_items, max_c, total);
    if (D == 128) {
        if (alike && total != 0ull) {
            T best = costs[0];
            r.p_all = 1;
            const int top = max_c / SPLIT_MIN_BLOCKS < SPLIT_MAX_PIECES ? max_c / SPLIT_MIN_BLOCKS : SPLIT_MAX_PIECES;
            for (int P = 2; P <= top; ++P)
                if (costs[P - 1] < best && (n_items > cus || n_items * P <= pmax)) { best = costs[P - 1]; r.p_all = P; }
        }
    }
    const auto granules = [&](int n) { return D == 128 ? n * 5 / 2 : n * (alike ? 12 : 4); };
    const int one = granules(CUS_PER_XCD), all = granules(cus) < pmax ? granules(cus) : pmax;
    r.g = all > one ? all : one;
    return r;
}

__device__ __forceinline__ int split_pieces(int c, unsigned long long total, const SplitRule& rule)
{
    if (total == 0ull) return 1;
    unsigned long long P = rule.p_all ? (unsigned long long)rule.p_all
                                      : (2ull * (unsigned)c * (unsigned)rule.g + total) / (2ull * total);
    const unsigned long long by_len = (unsigned)c / SPLIT_MIN_BLOCKS;
    if (P > by_len) P = by_len;
    if (P > (unsigned long long)SPLIT_MAX_PIECES) P = SPLIT_MAX_PIECES;
    return P < 1ull ? 1 : (int)P;
}

__global__ __launch_bounds__(1024) void plan_split_kernel(const int32_t* __restrict__ counts, int BH, int nb, int cap,
                                                          int pmax, int D, PlanRec* __restrict__ recs,
                                                          int32_t* __restrict__ arrived)
{
    __shared__ int hist[PLAN_BINS];              // by r = nb - length (r = 0: longest)
    __shared__ int ccache[PLAN_CACHE];           // counts of the first items, read once
    __shared__ int wave_sum[16];
    __shared__ unsigned long long total;          // kept key-blocks of this XCD's items
    __shared__ int longest;                       // of its rows
    __shared__ long long alike_cost[SPLIT_MAX_PIECES];
    const int x = blockIdx.x, tid = threadIdx.x;
    const int n_bh = (BH - x + XCDS - 1) / XCDS;
    const int n_items = n_bh > 0 ? n_bh * nb : 0;
    PlanRec* out = recs + (size_t)x * cap;
    auto item_of = [&](int i) { return ((i / nb) * XCDS + x) * nb + i % nb; };
    auto count_of = [&](int i) { return i < PLAN_CACHE ? ccache[i] : counts[item_of(i)]; };
    const PlanRec none = {-1, 0, 0, -1};
    for (int i = tid; i < pmax; i += 1024) arrived[(size_t)x * pmax + i] = 0;
    if (nb > PLAN_MAX_NB) {                       // no sort, no pieces: natural order
        for (int i = tid; i < cap; i += 1024) {
            PlanRec r = none;
            if (i < n_items) { r.item = item_of(i); r.nblk = counts[r.item]; }
            out[i] = r;
        }
        return;
    }
    if (tid == 0) { total = 0ull; longest = 0; }
#pragma unroll
    for (int j = 0; j < 8; ++j) hist[8 * tid + j] = 0;
    __syncthreads();
    {
        unsigned long long mine = 0ull;
        int mx = 0;
        for (int i = tid; i < n_items; i += 1024) {
            const int c = counts[item_of(i)];
            if (i < PLAN_CACHE) ccache[i] = c;
            mine += (unsigned long long)c;
            mx = c > mx ? c : mx;
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            mine += __shfl_down(mine, d, 64);
            const int o = __shfl_down(mx, d, 64);
            mx = o > mx ? o : mx;
        }
        if ((tid & 63) == 0) { atomicAdd(&total, mine); atomicMax(&longest, mx); }
    }
    for (int i = tid; i < cap; i += 1024) out[i] = none;
    __syncthreads();
    const unsigned long long tot = total;
    if (tid < SPLIT_MAX_PIECES) alike_cost[tid] = split_alike_cost<long long>(segment_cus(BH, nb, 128), n_items, longest, tid + 1);
    __syncthreads();
    const SplitRule rule = split_rule(D, segment_cus(BH, nb, 128), pmax, n_items, longest, tot, alike_cost);
    // partial-result slots in item order: thread t owns the items [lo, hi)
    const int per = (n_items + 1023) / 1024;
    const int lo = tid * per < n_items ? tid * per : n_items;
    const int hi = lo + per < n_items ? lo + per : n_items;
    int mine = 0;
    for (int i = lo; i < hi; ++i) {
        const int P = split_pieces(count_of(i), tot, rule);
        if (P > 1) mine += P;
    }
    const int first_slot = plan_block_scan(mine, wave_sum, tid);
    // pieces of item i: P (1 = whole) and the first partial slot
    auto pieces_of = [&](int c, int& run, int& P, int& slot0) {
        const int want = split_pieces(c, tot, rule);
        P = want;
        slot0 = -1;
        if (want > 1) {
            if (run + want <= pmax) slot0 = run; else P = 1;
            run += want;                          // the prefix counts every candidate
        }
    };
    {
        int run = first_slot;
        for (int i = lo; i < hi; ++i) {
            const int c = count_of(i);
            int P, slot0;
            pieces_of(c, run, P, slot0);
            for (int k = 0; k < P; ++k) atomicAdd(&hist[nb - (c * (k + 1) / P - c * k / P)], 1);
        }
    }
    __syncthreads();
    plan_scan_bins(hist, wave_sum, tid);
    {
        int run = first_slot;
        for (int i = lo; i < hi; ++i) {
            const int item = item_of(i);
            const int c = count_of(i);
            int P, slot0;
            pieces_of(c, run, P, slot0);
            for (int k = 0; k < P; ++k) {
                PlanRec r;
                r.item = item;
                r.blk0 = c * k / P;
                r.nblk = c * (k + 1) / P - r.blk0;
                r.w = (P > 1) ? (((x * pmax + slot0) << 8) | (k << 4) | (P - 1)) : -1;
                out[atomicAdd(&hist[nb - r.nblk], 1)] = r;
            }
        }
    }
}

// Up to SMALL_NB mask blocks per side: the plan in ONE launch, written for latency, from the mask itself or from counts
// that are there already.  The mask is read eight bytes per lane, all of an XCD's at once, and kept as one bit per
// block in LDS; a row's count is a population count of its stretch of bits.  The lists are not written here: an
// attention workgroup reads its own row of the mask (KeptBlocks).  Same rule and same records as plan_split_kernel and
// plan_kernel, in 32-bit arithmetic (the limits keep every intermediate below 2^32).
constexpr int SMALL_NB = 64;                     // mask blocks per side
constexpr int SMALL_PER_THREAD = 4;              // items of one XCD per thread, at most
constexpr int SMALL_ITEMS = 1024 * SMALL_PER_THREAD;
constexpr int SMALL_PIECES = 8192;               // pieces of eight mask bytes of one XCD's items

// eight mask bytes as eight bits
__device__ __forceinline__ unsigned byte_bits(unsigned lo, unsigned hi)
{
    auto four = [](unsigned v) {
        v |= v >> 4;
        v |= v >> 2;
        v |= v >> 1;
        return ((v & 0x01010101u) * 0x10204080u) >> 28;    // bit 8 i to bit 28 + i
    };
    return four(lo) | four(hi) << 4;
}

// PT items per thread, SWEEPS times 1024 pieces.
template <bool PIECES, int PT, int SWEEPS>
__global__ __launch_bounds__(1024) void plan_small_kernel(
    const unsigned char* __restrict__ mask, const int32_t* __restrict__ kv_lens, int kv_len, int N, int block,
    int H, int BH, int nb, int cap, int pmax, int D,
    int32_t* __restrict__ counts, int32_t* __restrict__ order, int32_t* __restrict__ arrived)
{
    __shared__ unsigned bits[1024 * SWEEPS / 4 + 4]; // pair g: one bit per mask block from byte g * pad on
    __shared__ int hist[SMALL_NB + 1], to[SMALL_NB + 1];    // by r = nb - length: records, and where the next one goes
    __shared__ int wave_sum[16], kept_sum[16], wave_max[16];
    __shared__ unsigned alike_cost[SPLIT_MAX_PIECES];
    const int x = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int n_bh = BH > x ? (BH - x + XCDS - 1) / XCDS : 0;
    const int n_items = n_bh * nb;
    const unsigned per_bh = (unsigned)(nb * nb);
    const unsigned ppb = (per_bh + 7u) / 8u, pad = (ppb + 3u) & ~3u;    // pieces of a pair, and their bytes of bits
    PlanRec* out = (PlanRec*)order + (size_t)x * cap;
    int32_t* ids = order + (size_t)x * cap;
    // f / ppb for f < 2^13 and i / nb for i < 2^12, nb <= 64, by 24-bit multiplications: with m = ceil(2^19 / d) the
    // quotient is exact as long as f * (m * d - 2^19) < 2^19, and m * d - 2^19 < d <= 2^6; ppb goes up to 2^9, whose
    // quotients come from one 32-bit multiplication (2^13 * 2^9 < 2^32; ppb = 1: the product wraps, handled apart)
    const unsigned magic_p = 0xffffffffu / ppb + 1u, magic_nb = ((1u << 19) + (unsigned)nb - 1u) / (unsigned)nb;
    auto div_p = [&](unsigned f) { return ppb == 1u ? f : __umulhi(f, magic_p); };
    auto div_nb = [&](unsigned f) { return __umul24(f, magic_nb) >> 19; };

    int c[PT], item[PT];
    int live[PT];                                // key-blocks that start below the valid length
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        const unsigned i = (unsigned)tid + 1024u * k, in = i < (unsigned)n_items ? i : 0u;
        const unsigned g = div_nb(in);
        item[k] = (int)(__umul24(g * XCDS + x, nb) + (in - __umul24(g, nb)));
        c[k] = 0;
        live[k] = kv_len;
        if (1024 * k < n_items) {                 // the same for the whole workgroup
            if (mask == nullptr) c[k] = counts[item[k]];
            else if (kv_lens != nullptr) live[k] = kv_lens[(int)(g * XCDS + x) / H];
        }
    }
    if (mask != nullptr) {
        const unsigned total = (unsigned)n_bh * ppb;
        unsigned lo[SWEEPS], hi[SWEEPS];
#pragma unroll
        for (int t = 0; t < SWEEPS; ++t) {
            lo[t] = hi[t] = 0u;
            if (1024u * t < total) {              // the same for the whole workgroup
                // lanes past the end load the last piece again, so that no load sits behind a branch; the last piece
                // of a pair ends with it: what belongs to the piece before is shifted out
                const unsigned f = (unsigned)tid + 1024u * t, fc = f < total ? f : total - 1u;
                const unsigned g = div_p(fc), r = (fc - __umul24(g, ppb)) * 8u;
                const unsigned char* src = mask + (size_t)(g * XCDS + x) * per_bh;
                if (nb >= 3) {
                    const unsigned over = r + 8u > per_bh ? r + 8u - per_bh : 0u;
                    unsigned long long v;
                    __builtin_memcpy(&v, src + (r - over), 8);
                    v >>= 8u * over;
                    lo[t] = (unsigned)v;
                    hi[t] = (unsigned)(v >> 32);
                } else {
                    for (unsigned e = 0; e < per_bh; ++e) lo[t] |= (unsigned)src[e] << (8u * e);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < SWEEPS; ++t) {
            const unsigned f = (unsigned)tid + 1024u * t;
            if (f < total) {
                const unsigned g = div_p(f);
                ((unsigned char*)bits)[__umul24(g, pad) + (f - __umul24(g, ppb))] = (unsigned char)byte_bits(lo[t], hi[t]);
            }
        }
    }
    if (tid <= SMALL_NB) hist[tid] = 0;
    __syncthreads();

    int kept = 0, longest = 0;
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        const unsigned i = (unsigned)tid + 1024u * k;
        const bool has = i < (unsigned)n_items;
        if (mask != nullptr && 1024 * k < n_items) {
            const unsigned in = has ? i : 0u, g = div_nb(in), at = __umul24(in - __umul24(g, nb), nb), w = (g * pad >> 2) + (at >> 5);
            const unsigned long long b = ((unsigned long long)bits[w + 1] << 32) | bits[w], up = bits[w + 2];
            const unsigned s = at & 31u;
            const unsigned long long row = s ? (b >> s) | (up << (64u - s)) : b;
            int len = live[k];
            len = len < 0 ? 0 : (len > N ? N : len);
            const int blocks = (len + block - 1) / block;
            const int cols = blocks < nb ? blocks : nb;
            c[k] = __popcll(row & (cols >= 64 ? ~0ull : (1ull << cols) - 1ull));
        }
        if (!has) c[k] = 0;
        if (has && mask != nullptr) counts[item[k]] = c[k];
        kept += c[k];
        longest = c[k] > longest ? c[k] : longest;
    }
    unsigned tot = 0u;                            // kept key-blocks of this XCD's items
    int P[PT], slot0[PT];
#pragma unroll
    for (int k = 0; k < PT; ++k) { P[k] = 1; slot0[k] = -1; }
    if constexpr (PIECES) {
        const int sum = wave_scan_inclusive(kept);
        longest = wave_max_to_last(longest);
        if (lane == 63) { kept_sum[tid >> 6] = sum; wave_max[tid >> 6] = longest; }
        __syncthreads();
        longest = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) { tot += (unsigned)kept_sum[w]; longest = wave_max[w] > longest ? wave_max[w] : longest; }
        if (D == 128 && rows_alike(n_items, longest, tot)) {   // the same for the whole workgroup
            if (tid < SPLIT_MAX_PIECES) alike_cost[tid] = split_alike_cost<unsigned>(segment_cus(BH, nb, 128), n_items, longest, tid + 1);
            __syncthreads();
        }
        const SplitRule rule = split_rule(D, segment_cus(BH, nb, 128), pmax, n_items, longest, tot, alike_cost);
        int want[PT], mine = 0;
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            want[k] = 1;
            if (1024 * k < n_items && tot != 0u) {
                unsigned n = rule.p_all ? (unsigned)rule.p_all : (2u * (unsigned)c[k] * (unsigned)rule.g + tot) / (2u * tot);
                const unsigned by_len = (unsigned)c[k] / SPLIT_MIN_BLOCKS;
                n = n > by_len ? by_len : n;
                n = n > (unsigned)SPLIT_MAX_PIECES ? SPLIT_MAX_PIECES : n;
                want[k] = n < 1u ? 1 : (int)n;
            }
            mine += want[k] > 1 ? want[k] : 0;
        }
        // slots: a scan inside each wavefront, then the totals of the wavefronts before
        const int incl = wave_scan_inclusive(mine);
        if (lane == 63) wave_sum[tid >> 6] = incl;
        __syncthreads();
        int run = incl - mine;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int t = wave_sum[w];
            run += w < tid >> 6 ? t : 0;
        }
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            if (want[k] > 1) {
                if (run + want[k] <= pmax) { slot0[k] = run; P[k] = want[k]; }
                run += want[k];                   // the prefix counts every candidate
            }
        }
    }
    // piece j holds c(j+1)/P - cj/P key-blocks: c/P, plus one whenever the running remainder wraps
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        if ((unsigned)tid + 1024u * k < (unsigned)n_items) {
            if (!PIECES || P[k] == 1) {
                atomicAdd(&hist[nb - c[k]], 1);
            } else {
                const int q = c[k] / P[k], r = c[k] - q * P[k];
                int e = 0;
                for (int j = 0; j < P[k]; ++j) {
                    e += r;
                    const int extra = e >= P[k];
                    e -= extra ? P[k] : 0;
                    atomicAdd(&hist[nb - (q + extra)], 1);
                }
            }
        }
    }
    __syncthreads();
    const int mine = lane < nb ? hist[lane] : 0, upto = wave_scan_inclusive(mine);
    const int longer = __builtin_amdgcn_readlane(upto, 63), n_rec = longer + hist[nb];
    if (tid < nb) to[tid] = upto - mine;          // (nb <= 64: wavefront 0)
    if (tid == 0) to[nb] = longer;
    __syncthreads();
    // At launch the dispatcher deals the XCD's workgroups out to its 32 CUs in turn (seen in
    // the hardware ids of traced launches): CU i starts with the records i, i + 32, ...
    // Longest-first order would give CU 0 the longest record of every round of 32, so the second
    // and the fourth round of the first wave (as many records as the XCD has places) run backwards.
    // Later records go wherever a place frees up first and stay longest first.
    const int cus = PIECES ? segment_cus(BH, nb, 128) : CUS_PER_XCD;      // records of a round (few pairs of up to 64 64-token blocks: no plan)
    auto place = [&](int len) {
        int pos = atomicAdd(&to[nb - len], 1);
        const int first = pos < 3 * cus ? cus : 3 * cus, at = pos - first;    // of the second, of the fourth round
        if (at >= 0 && at < cus && (first == cus || (PIECES && D == 64))) {
            const int left = n_rec - first;
            pos = first + (left < cus ? left : cus) - 1 - at;
        }
        return pos;
    };
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        if ((unsigned)tid + 1024u * k < (unsigned)n_items) {
            if constexpr (!PIECES) {
                ids[place(c[k])] = item[k];
            } else if (P[k] == 1) {
                const PlanRec rec = {item[k], 0, c[k], -1};
                out[place(c[k])] = rec;
            } else {
                const int q = c[k] / P[k], r = c[k] - q * P[k];
                int e = 0, b0 = 0;
                for (int j = 0; j < P[k]; ++j) {
                    e += r;
                    const int extra = e >= P[k];
                    e -= extra ? P[k] : 0;
                    const PlanRec rec = {item[k], b0, q + extra, ((x * pmax + slot0[k]) << 8) | (j << 4) | (P[k] - 1)};
                    b0 += rec.nblk;
                    out[place(rec.nblk)] = rec;
                }
            }
        }
    }
    if constexpr (PIECES) {
        const PlanRec none = {-1, 0, 0, -1};
        for (int i = n_rec + tid; i < cap; i += 1024) out[i] = none;
        for (int i = tid; i < pmax; i += 1024) arrived[(size_t)x * pmax + i] = 0;
    } else {
        for (int i = n_rec + tid; i < cap; i += 1024) ids[i] = -1;
    }
}

// ---------------------------------------------------------------------------
// Attention.  D in {64,128}; NW wavefronts; query tile = 32*NW rows.
// ---------------------------------------------------------------------------
// LDS tile geometry.  A 64 x D bf16 tile is stored row-major WITHOUT padding, because
// it is filled by direct global->LDS loads (global_load_lds_dwordx4: one instruction
// writes 64 lanes x 16 B = 1 KB of consecutive LDS).  Bank conflicts are avoided by
// permuting the 16-byte chunks inside each row: physical chunk = logical chunk ^ swz(row).
// The permutation is applied on the global side of the copy (each lane chooses which
// chunk of the row it fetches), so the copy stays fully coalesced.
template <int D>
struct Geo {
    static constexpr int ROW_BYTES = D * 2;                 // 256 | 128
    static constexpr int CPR = D / 8;                       // chunks per row: 16 | 8
    static constexpr int TILE_BYTES = KT * ROW_BYTES;       // 16384 | 8192
    static constexpr int ROWS_PER_LOAD = 1024 / ROW_BYTES;  // 4 | 8
    static constexpr int LOADS = TILE_BYTES / 1024;         // 16 | 8
    // (The swizzles are those of attn_sparse_sg_kernel<64>; the stream has its own.)
    // K is read 16 bytes per lane, lanes = consecutive rows at one logical chunk:
    // 16 consecutive rows must land on 16 different chunks of the 256-byte bank line.
    static __device__ __forceinline__ int swz_k(int row) { static_assert(D == 64, ""); return (row >> 1) & 7; }
    // V is read by the transpose read as 4-row x 64-byte patches: consecutive rows must
    // land on different 64-byte groups of the bank line.
    static __device__ __forceinline__ int swz_v(int row) { static_assert(D == 64, ""); return ((row >> 1) & 1) << 2; }
};

// Issue the asynchronous copy of rows key0..key0+63 of `src` into an LDS tile.  Rows at or
// beyond kv_len are replaced by row kv_len-1 (finite data; their probabilities are exactly
// 0, and their scores are overwritten with -inf, so they never contribute).
template <int D, int NW, bool IS_V>
__device__ __forceinline__ void issue_tile(const Rows& src, int key0, int kv_len,
                                           char* lds, int wave, int lane)
{
    typedef Geo<D> G;
    constexpr int PER_WAVE = G::LOADS / NW;
    // global_load_lds_dwordx4: LDS address = M0 + offset + 16 * lane, memory address + the same offset.  Written as
    // assembly so that the copy pipeline is ordered only by the explicit vmcnt waits and barriers of the main loop
    // (the compiler would otherwise wait for all copies before LDS reads it cannot disambiguate).  M0 has no other
    // user in these kernels.  A copy may not be the next instruction after the scalar write of M0 (one wait state)
    // and the compiler does not look into assembly for that: s_nop 0, under 1 % (two copies behind one M0: 0.7 % slower).
    const int ld0 = wave * PER_WAVE;                        // wave-uniform
    auto row_of = [&](int i) { return (ld0 + i) * G::ROWS_PER_LOAD + lane / G::CPR; };
    auto chunk_of = [&](int i) { return (unsigned)((lane % G::CPR) ^ (IS_V ? G::swz_v(row_of(i)) : G::swz_k(row_of(i)))) * 16u; };
    auto dst = [&](int i) { return (unsigned)(size_t)LDS_PTR(char, lds + (ld0 + i) * 1024); };
    if (key0 + KT <= kv_len) {
        // whole tile valid: scalar tile base + a per-lane byte offset that does not depend
        // on the tile (no vector arithmetic per copy)
        const char* tile = src.row(key0);                  // a tile never straddles the segments
        auto off = [&](int i) { return (unsigned)row_of(i) * src.row_bytes + chunk_of(i); };
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i)
            asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(dst(i)), "v"(off(i)), "s"(tile));
    } else {
        auto at = [&](int i) {
            int grow = key0 + row_of(i);
            grow = grow < kv_len ? grow : kv_len - 1;
            return (key0 < src.n0 ? src.base0 : src.base1) + (size_t)grow * src.row_bytes + chunk_of(i);
        };
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i)
            asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"{m0}"(dst(i)), "v"(at(i)));
    }
}

// The same copy, one instruction at a time, as buffer loads: rows at or beyond kv_len (and whole
// tiles there) lie outside the buffer and arrive as zeros, so nothing in the tile loop branches on
// the tile.  A descriptor covers the valid part of one tile.
typedef int i32x4 __attribute__((ext_vector_type(4)));
struct TileBuffer {
    unsigned lo, hi, bytes;
};
template <int ROWS>
__device__ __forceinline__ TileBuffer tile_buffer(const Rows& src, int key0, int kv_len)
{
    const char* tile = src.row(key0);                      // a tile never straddles the segments
    int rows = kv_len - key0;
    rows = rows < 0 ? 0 : rows;
    asm("" : "+s"(rows));                                  // two scalar instructions, not one vector clamp
    rows = rows > ROWS ? ROWS : rows;
    TileBuffer r;
    r.lo = (unsigned)(size_t)tile;
    r.hi = (unsigned)((size_t)tile >> 32) & 0xffffu;
    r.bytes = (unsigned)rows * src.row_bytes;
    return r;
}
// The descriptor of a run of tiles moved on by one.
__device__ __forceinline__ void next_tile_of(TileBuffer& b, unsigned tile_bytes)
{
    const unsigned long long at = ((unsigned long long)b.hi << 32 | b.lo) + tile_bytes;
    b.lo = (unsigned)at;
    b.hi = (unsigned)(at >> 32);
    unsigned left = b.bytes - tile_bytes;
    asm("" : "+s"(left));                                  // (a saturating subtraction would be a vector instruction)
    b.bytes = b.bytes > tile_bytes ? left : 0u;
}
// One copy, or two whose second KB is in the next KB of the stage, behind one write of M0 (see issue_tile).
__device__ __forceinline__ void copy_1k(const TileBuffer& b, unsigned off, unsigned dst)
{
    const i32x4 rsrc = {(int)b.lo, (int)b.hi, (int)b.bytes, 0x00020000};
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"{m0}"(dst), "v"(off), "s"(rsrc));
}
__device__ __forceinline__ void copy_2k(const TileBuffer& b, unsigned off, unsigned off_next, unsigned dst)
{
    const i32x4 rsrc = {(int)b.lo, (int)b.hi, (int)b.bytes, 0x00020000};
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %3, 0 offen lds\n\tbuffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds"
                 ::"{m0}"(dst), "v"(off), "v"(off_next - 1024u), "s"(rsrc));    // (a row is at least D elements: not negative)
}

struct SoftmaxState {
    float m;      // reference of the exponents, in units of scale * log2(e); same in both lane halves
    float l;      // this lane's partial sum of probabilities
};

// ---------------------------------------------------------------------------
// The matrix work of one tile as a stream of ITEMS.  An item is one MFMA together with
// the LDS read(s) of its A operand:
//   items 0 .. NPV-1     O^T += V^T P^T   item = (g, db): 16-key group g = 2 rb + t, 32-row
//                        block db of O^T; two transpose reads (keys 4h+r and 8+4h+r)
//   items NPV .. NI-1    S^T += K Q^T     item = (t, rb): k-step t, 32-key row block rb;
//                        one 128-bit read
// The reads of item i+PD are requested before the MFMA of item i is issued, so every
// operand has PD MFMAs (about 200 cycles) of lead.  The reads are inline assembly with
// their own s_waitcnt: issued through compiler builtins the transpose reads carry no
// alias scope and each of them would wait for ALL outstanding global->LDS copies.  LDS
// returns data in order, so "lgkmcnt(N)" = everything but the newest N requests has
// arrived; the counter has 4 bits, which bounds PD (at most 15 requests in flight).
// ---------------------------------------------------------------------------
template <int D, int PD_>
struct TileItems {
    static constexpr int DB = D / 32, KS = D / 16;
    static constexpr int NPV = 4 * DB;
    static constexpr int NQK = 2 * KS;
    static constexpr int NI = NPV + NQK;
    static constexpr int PD = PD_;             // how many items ahead the LDS reads are requested
    static constexpr int NBUF = PD + 1;
    static constexpr int reads(int i) { return i < NPV ? 2 : 1; }
    // LDS requests of the items after i that are in flight while item i is awaited
    static constexpr int newer(int i, int last)
    {
        int s = 0;
        for (int k = i + 1; k <= i + PD && k < last; ++k) s += reads(k);
        return s;
    }
};

template <int D, int PD>
struct TileCtx {
    unsigned vaddr[D / 32];                    // LDS byte address of this lane's transpose-read patch, per O^T block
    unsigned kbase;                            // LDS byte address of row n of the K tile
    unsigned kxor;                             // (h ^ swz_k(n)) << 4: chunk (2t+h) ^ swz == (2t) ^ (kxor >> 4)
    u32x2 lo[TileItems<D, PD>::NBUF];              // item i lives in slot i % NBUF
    u32x2 hi[TileItems<D, PD>::NBUF];
    u32x4 kf[TileItems<D, PD>::NBUF];
};

template <int D, int PD, int I>
__device__ __forceinline__ void item_request(TileCtx<D, PD>& c)
{
    typedef TileItems<D, PD> TI;
    constexpr int RB = Geo<D>::ROW_BYTES;
    constexpr int slot = I % TI::NBUF;
    if constexpr (I < TI::NPV) {
        constexpr int g = I / TI::DB, db = I % TI::DB;
        constexpr int row0 = (g >> 1) * 32 + (g & 1) * 16;
        asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                     : "=&v"(c.lo[slot]), "=&v"(c.hi[slot])
                     : "v"(c.vaddr[db]), "i"(row0 * RB), "i"((row0 + 8) * RB));
    } else {
        constexpr int t = (I - TI::NPV) / 2, rb = (I - TI::NPV) % 2;
        const unsigned ka = c.kbase + ((unsigned)(t << 5) ^ c.kxor);
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(c.kf[slot]) : "v"(ka), "i"(rb * 32 * RB));
    }
}

// Wait for item I; LAST = end of the run of items whose requests may be in flight.  The
// fragment is an in/out operand so that its use is ordered after the wait.
template <int D, int PD, int I, int LAST>
__device__ __forceinline__ void item_wait(TileCtx<D, PD>& c)
{
    typedef TileItems<D, PD> TI;
    constexpr int slot = I % TI::NBUF;
    constexpr int N = TI::newer(I, LAST);
    static_assert(N + TI::reads(I) <= 15, "lgkmcnt is a 4-bit counter");
    if constexpr (I < TI::NPV) asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(c.lo[slot]), "+v"(c.hi[slot]) : "i"(N));
    else asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(c.kf[slot]) : "i"(N));
}

template <int D, int PD, int I>
__device__ __forceinline__ void item_mfma(const TileCtx<D, PD>& c, const bf16x8 (&pb)[4], const bf16x8 (&qf)[D / 16],
                                          f32x16 (&acc)[D / 32], f32x16 (&st)[2])
{
    typedef TileItems<D, PD> TI;
    constexpr int slot = I % TI::NBUF;
    if constexpr (I < TI::NPV) {
        constexpr int g = I / TI::DB, db = I % TI::DB;
        const u32x4 both = __builtin_shufflevector(c.lo[slot], c.hi[slot], 0, 1, 2, 3);
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pb[g], acc[db], 0, 0, 0);
    } else {
        constexpr int t = (I - TI::NPV) / 2, rb = (I - TI::NPV) % 2;
        f32x16 cin = st[rb];
        if constexpr (t == 0) {                            // first k-step starts from zero
#pragma unroll
            for (int j = 0; j < 16; ++j) cin[j] = 0.f;
        }
        st[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, c.kf[slot]), qf[t], cin, 0, 0, 0);
    }
}

// Request the first PD items of the run [FROM, TO).
template <int D, int PD, int FROM, int TO, int I = FROM>
__device__ __forceinline__ void items_prefetch(TileCtx<D, PD>& c)
{
    if constexpr (I < TO && I < FROM + PD) {
        item_request<D, PD, I>(c);
        items_prefetch<D, PD, FROM, TO, I + 1>(c);
    }
}

// Issue items [I, TO); items_prefetch<D, PD, I, TO> must have been called before.
template <int D, int PD, int I, int TO>
__device__ __forceinline__ void items_run(TileCtx<D, PD>& c, const bf16x8 (&pb)[4], const bf16x8 (&qf)[D / 16],
                                          f32x16 (&acc)[D / 32], f32x16 (&st)[2])
{
    if constexpr (I < TO) {
        if constexpr (I + PD < TO) item_request<D, PD, I + PD>(c);
        item_wait<D, PD, I, TO>(c);
        item_mfma<D, PD, I>(c, pb, qf, acc, st);
        items_run<D, PD, I + 1, TO>(c, pb, qf, acc, st);
    }
}

// Lane addresses for the tile held in (lds_k, lds_v).
//   K: lane (n, h) reads row n (+32 rb), logical chunk 2t + h of k-step t.
//   V: within a 16-lane group, lane j points at row j/4, columns 4 (j%4)..+3 of a 4 x 16
//      patch of the transpose read and lane i receives column i; lane half h covers rows +4h.
template <int D, int PD>
__device__ __forceinline__ void k_addresses(const char* lds_k, int n, int h, TileCtx<D, PD>& c)
{
    typedef Geo<D> G;
    c.kbase = (unsigned)(size_t)LDS_PTR(const char, lds_k) + n * G::ROW_BYTES;
    c.kxor = (unsigned)(h ^ G::swz_k(n)) << 4;
}

template <int D>
__device__ __forceinline__ void v_addresses(const char* lds_v, int h, int tr_row, int tr_col, unsigned (&vaddr)[D / 32])
{
    typedef Geo<D> G;
    const unsigned vbase = (unsigned)(size_t)LDS_PTR(const char, lds_v) + (4 * h + tr_row) * G::ROW_BYTES + tr_col * 2;
    const int vx = G::swz_v(tr_row) >> 2;                  // 64-byte group swizzle of this lane's rows
#pragma unroll
    for (int db = 0; db < D / 32; ++db) vaddr[db] = vbase + ((db ^ vx) << 6);
}

// Keys at or beyond kv_len -> -inf.  Register i of row block rb of S^T holds key
// key0 + 32 rb + 8 (i/4) + 4 h + i%4  of query n.
__device__ __forceinline__ void mask_tail(f32x16 (&st)[2], int key0, int kv_len, int h)
{
    if (__builtin_expect(key0 + KT > kv_len, 0)) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int key = key0 + 32 * rb + 8 * (i >> 2) + 4 * h + (i & 3);
                if (key >= kv_len) st[rb][i] = -INFINITY;
            }
    }
}

// Online softmax of one tile (one query per lane; the two lane halves hold disjoint keys).
// Probabilities are exp2(c * s - m) with c = scale * log2(e) and a per-query reference m (kept in
// exponent units); any m gives the same quotient acc / l, and bf16 and fp32 share their exponent
// range, so m need not be the running maximum.  No maximum on the common path: m comes from the first tile and
// moves only when a later tile's probabilities get large: their sum, which is needed anyway, exceeds 2^60 (or is not
// a number).  Then the tile's maximum becomes the reference and the tile's probabilities are computed again.
// When m moves, l and the accumulators are rescaled.  Leaves the probabilities as bf16 MFMA
// operands: pb[2 rb + t] = keys 16t + {4h..4h+3, 8+4h..8+4h+3} of row block rb.
template <int D>
__device__ __forceinline__ void softmax_tile(const f32x16 (&st)[2], f32x16 (&acc)[D / 32], SoftmaxState& st_,
                                             float c, bool first, bf16x8 (&pb)[4])
{
    constexpr int DB = D / 32;
    // The row sum adds up the probabilities two per instruction (v_dot2 of the bf16 pair against
    // 1.0): it is then over the probabilities as rounded to bf16, the weights the PV product applies.
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 ones;
    ones[0] = (__bf16)1.0f;
    ones[1] = (__bf16)1.0f;
    auto probabilities = [&]() -> float {
        float rs0 = 0.f, rs1 = 0.f;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int rb = g >> 1, t = g & 1;
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
                bf16x2 pr;
                pr[0] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(st[rb][8 * t + i], c, -st_.m));
                pr[1] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(st[rb][8 * t + i + 1], c, -st_.m));
                pb[g][i] = pr[0];
                pb[g][i + 1] = pr[1];
                if (i & 2) rs1 = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rs1, false);
                else rs0 = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, rs0, false);
            }
        }
        return rs0 + rs1;
    };
    // the tile's largest exponent relative to m (on the first tile: the exponent itself)
    auto tile_max = [&]() -> float {
        float mx = fmaxf(st[0][0], st[1][0]);
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(fmaxf(mx, st[0][i]), st[1][i]);
        auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        return first ? mx * c : __builtin_fmaf(mx, c, -st_.m);
    };
    float rs = 0.f, mx = 0.f;
    bool move = first;
    if (!first) {
        rs = probabilities();
        move = __builtin_amdgcn_ballot_w64(!(rs <= 0x1p60f)) != 0ull;     // also true for inf and NaN
    }
    if (move) {
        mx = tile_max();
        // mx is finite: every visited tile has a valid key.  On the first tile nothing has been
        // accumulated yet; later the reference only moves up.
        const float delta = first ? mx : fmaxf(mx, 0.f);
        const float alpha = first ? 1.0f : __builtin_amdgcn_exp2f(-delta);
        st_.m = first ? mx : st_.m + delta;
        st_.l *= alpha;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[i][j] *= alpha;
        rs = probabilities();
    }
    st_.l += rs;
}

// Epilogue: O = acc / l as bf16.  Register 4j+r of block db holds d = 32 db + 8 j + 4 h + r
// of this lane's query; rows at or beyond kv_len and rows without any kept key become 0.
template <int D>
__device__ __forceinline__ void write_output(const Rows& O, const f32x16 (&acc)[D / 32], float l_part,
                                             int qrow, bool qvalid, int N, int h)
{
    float l_run = l_part;
    {
        auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
        l_run = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
    const float inv = (qvalid && l_run > 0.f) ? 1.0f / l_run : 0.f;
    if (qrow < N) {
        __bf16* orow = (__bf16*)const_cast<char*>(O.row(qrow));
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                bf16x4 ov;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = acc[db][4 * j + r] * inv;
                    ov[r] = (__bf16)((inv != 0.f) ? x : 0.f);
                }
                *(bf16x4*)(orow + 32 * db + 8 * j + 4 * h) = ov;
            }
    }
}

// Q^T fragments (B operand of S^T = K Q^T): lane (n, h) holds Q[qrow][16t + 8h .. +8].  Requested by explicit
// assembly: the compiler then places no waits of
// its own for them (it cannot count the tile copies issued around them and would wait for
// everything); the caller waits with wait_vmcnt and then passes the fragments through
// q_arrived so that their uses stay behind that wait.  Rows that are not valid read row 0
// of the (sample, head) and are zeroed afterwards.
template <int D>
__device__ __forceinline__ void load_q_async(const Rows& Q, int qrow, bool qvalid, int h, u32x4 (&raw)[D / 16])
{
    const __bf16* src = (const __bf16*)Q.row(qvalid ? qrow : 0) + 8 * h;
#pragma unroll
    for (int t = 0; t < D / 16; ++t)
        asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=v"(raw[t]) : "v"(src), "i"(32 * t));
}

template <int D>
__device__ __forceinline__ void q_arrived(u32x4 (&raw)[D / 16], bool qvalid, bf16x8 (&qf)[D / 16])
{
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
        asm volatile("" : "+v"(raw[t]));
        const u32x4 zero = {0u, 0u, 0u, 0u};
        qf[t] = __builtin_bit_cast(bf16x8, qvalid ? raw[t] : zero);
    }
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt in
// bits 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at their maxima)
template <int VM>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(VM >= 0 && VM < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (VM & 15) | ((VM >> 4) << 14));
}

// Values computed from registers only carry no ordering against a barrier; an empty volatile
// assembly statement that "modifies" them makes them complete before whatever follows it.
__device__ __forceinline__ void pin_in_phase(bf16x8 (&pb)[4], float& l)
{
    u32x4 a = __builtin_bit_cast(u32x4, pb[0]), b = __builtin_bit_cast(u32x4, pb[1]);
    u32x4 c = __builtin_bit_cast(u32x4, pb[2]), d = __builtin_bit_cast(u32x4, pb[3]);
    asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(l));
    pb[0] = __builtin_bit_cast(bf16x8, a); pb[1] = __builtin_bit_cast(bf16x8, b);
    pb[2] = __builtin_bit_cast(bf16x8, c); pb[3] = __builtin_bit_cast(bf16x8, d);
}

// Workgroup barrier that is also a boundary for the instruction scheduler: register-only
// work (the softmax arithmetic) must not drift from its phase into the neighbouring one.
__device__ __forceinline__ void phase_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------
// The tile loop as ONE software-pipelined stream of 16x16x32 MFMAs.  A wavefront owns NQ groups of
// 16 queries; a step = 32 keys.  Step i issues
//   items 0 .. NQK-1     S_{i+1}^T = K_{i+1} Q^T     per item: one 128-bit LDS read, NQ MFMAs
//   items NQK .. NI-1    O^T += V_i^T P_i^T          per item: two LDS transpose reads, NQ MFMAs
// and between the MFMAs, a few instructions at a time, the softmax arithmetic that needs no MFMA of
// this half: the second half of step i's probabilities beside the first items, the first half of
// step i+1's beside the others.  The LDS reads of an item are requested PD items ahead, across the
// end of a step.
// What bounds it and why this form.  A full chip lowers its clock under this load (from 2.4 GHz to 2.11 at N = 4608 and
// 1.82 at N = 16896, D = 128, with the matrix pipe busy 57 and 72 % of the cycles), so energy per product counts as much
// as cycles: on unit-normal data a loop of nothing but 32x32x16 MFMAs sustains 1.65 PFLOP/s, of 16x16x32 ones 1.82
// (mfma_probe.hip).  The row sum is an MFMA of ones: 2-3 % of the call faster than v_dot2 beside the MFMAs, and that 5 %
// faster than vector adds.  Dense B = 1, H = 24, D = 128, against softmax and MFMA phases alternating between two groups
// of wavefronts: N = 4608 242 -> 218 us (1.20 PFLOP/s), N = 16896 3166 -> 2689 us (1.30); D = 64, B = 2, N = 4480
// 278 -> 231 us.  At D = 64 (B = 8, N = 4480) the vector port is busy 68 % of the cycles, two fifths of that with
// exponentials, all issue ports together 86 %, the matrix pipe 60 %.
// Layouts (lane = 16 g + n):
//   K, V^T operand   lane holds row n of the 16-row fragment, its 8 elements 8 g .. 8 g + 7 of 32
//   S^T              register r of tile kt, group q: key 16 kt + 4 g + r, query 16 q + n
//   P^T operand      the 8 probabilities of a lane and query group, tile 0 then tile 1, as bf16: the
//                    contraction index 8 g + e stands for key 16 (e / 4) + 4 g + e % 4, and V^T is
//                    fetched in that order
// ---------------------------------------------------------------------------
template <int D, int NQ_, int PD_, int NBUF_, int UP_, int UP_AGAIN_>
struct Stream {
    static constexpr int NQ = NQ_;
    static constexpr float UP = UP_, UP_AGAIN = UP_AGAIN_;     // see soft_close
    static constexpr int KS = D / 32;          // k-steps of a score
    static constexpr int DT = D / 16;          // 16-row blocks of O^T
    static constexpr int NQK = 2 * KS, NPV = DT, NI = NQK + NPV;
    static constexpr int PD = PD_, NBUF = NBUF_;
    static constexpr int HALF = 2 * NQ;        // pairs of probabilities in half a step
    static constexpr int UNITS = NQK * NQ;     // MFMAs in half a step
    static constexpr int UPM = 4 * HALF / UNITS;    // quarter pairs beside one MFMA: 1 at D = 128, 2 at D = 64
    static_assert(NQK == NPV && UPM * UNITS == 4 * HALF && (UPM == 1 || UPM == 2), "");
    static_assert(NBUF > PD && NI % NBUF == 0, "an item keeps its buffer from step to step");
    static constexpr int reads(int i) { return (i % NI) < NQK ? 1 : 2; }
    // LDS requests newer than item i's when everything before item `last` has been requested
    static constexpr int newer(int i, int last)
    {
        int s = 0;
        for (int k = i + 1; k < last; ++k) s += reads(k);
        return s;
    }
    // LDS tile geometry: as Geo, with the chunks of a V row swizzled for 16-row x 32-byte patches
    static constexpr int RB = D * 2;
    static __device__ __forceinline__ int swz_k(int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); }
    static __device__ __forceinline__ int swz_v(int row) { return D == 128 ? ((row & 7) << 1) : (((row >> 1) & 3) << 1); }
};

template <class S, int D>
struct StreamRegs {
    unsigned kaddr[S::KS];                     // LDS byte address of this lane's chunk of K row n, per k-step
    unsigned vaddr[S::DT];                     // of its element of the transpose read, per block of O^T
    u32x2 lo[S::NBUF], hi[S::NBUF];
    u32x4 kf[S::NBUF];
    bf16x8 qf[S::NQ][S::KS];
    f32x16 acc[S::DT * S::NQ / 4];             // block b, query group q: registers of quarter b * NQ + q
    f32x4 ls[S::NQ];                           // row sums, the same in all four registers
    float m[S::NQ];                            // references of the exponents
    bf16x8 ones;                               // 1.0 everywhere
    unsigned seen;                             // all packed probabilities since the references last moved, or-ed
    float x0, x1, e0, e1;                      // pairs under way
};

constexpr float REF_LOWEST = -1e30f;           // of a query whose first step has no finite score

// Lane addresses in a K tile at byte address k0 and a V tile at v0.
template <class S, int D>
__device__ __forceinline__ void stream_addresses(StreamRegs<S, D>& x, unsigned k0, unsigned v0, int lane)
{
    const int n = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < S::KS; ++t) x.kaddr[t] = k0 + n * S::RB + (((4 * t + g) ^ S::swz_k(n)) << 4);
    // 16 lanes of a group: lane j points at row 4 g + j / 4, columns 4 (j % 4) .. + 3 of the block
    const int row = 4 * g + (n >> 2);
#pragma unroll
    for (int b = 0; b < S::DT; ++b)
        x.vaddr[b] = v0 + row * S::RB + (((2 * b + ((n & 3) >> 1)) ^ S::swz_v(row)) << 4) + (n & 1) * 8;
}

// Request item I (I >= NI: item I - NI of the next step); KC, KN, VC: byte offsets of the 32 rows
// of K_{i+1}, K_{i+2} and V_i from the addresses of the context.
template <class S, int D, int KC, int KN, int VC, int I>
__device__ __forceinline__ void stream_request(StreamRegs<S, D>& x)
{
    constexpr int J = I % S::NI, slot = J % S::NBUF;
    if constexpr (J < S::NQK) {
        constexpr int t = J / 2, kt = J % 2;
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(x.kf[slot]) : "v"(x.kaddr[t]), "i"((I < S::NI ? KC : KN) + kt * 16 * S::RB));
    } else {
        asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                     : "=&v"(x.lo[slot]), "=&v"(x.hi[slot])
                     : "v"(x.vaddr[J - S::NQK]), "i"(VC), "i"(VC + 16 * S::RB));
    }
}

// Wait for item I when everything before item LAST has been requested.
template <class S, int D, int I, int LAST>
__device__ __forceinline__ void stream_wait(StreamRegs<S, D>& x)
{
    constexpr int slot = I % S::NBUF, N = S::newer(I, LAST);
    static_assert(N + S::reads(I) <= 15, "lgkmcnt is a 4-bit counter");
    if constexpr (I % S::NI < S::NQK) asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x.kf[slot]) : "i"(N));
    else asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(x.lo[slot]), "+v"(x.hi[slot]) : "i"(N));
}

// The requests of a step that does not exist are in flight when the loop ends: they land before
// their registers serve anything else.
template <class S, int D>
__device__ __forceinline__ void stream_drain(StreamRegs<S, D>& x)
{
    asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
    for (int b = 0; b < S::NBUF; ++b) asm volatile("" : "+v"(x.kf[b]));
}

// Four 16x16x32 accumulators live in one 16-register vector: the compiler then updates a quarter in
// place.  (As vectors of their own they move to other registers with every product, and the second
// set of registers spills.)
template <int Q>
__device__ __forceinline__ f32x4 quarter(const f32x16& v)
{
    return __builtin_shufflevector(v, v, 4 * Q, 4 * Q + 1, 4 * Q + 2, 4 * Q + 3);
}
template <int Q>
__device__ __forceinline__ void set_quarter(f32x16& v, f32x4 x)
{
    v[4 * Q] = x[0]; v[4 * Q + 1] = x[1]; v[4 * Q + 2] = x[2]; v[4 * Q + 3] = x[3];
}
template <int Q>
__device__ __forceinline__ void mfma16(f32x16& acc, bf16x8 a, bf16x8 b, bool zero = false)
{
    const f32x4 none = {0.f, 0.f, 0.f, 0.f};
    set_quarter<Q>(acc, __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, zero ? none : quarter<Q>(acc), 0, 0, 0));
    asm volatile("" : "+v"(acc));                 // in place
}

// S^T of one step: tile kt, query group q
template <class S>
struct Scores {
    f32x16 v[(S::NQ + 1) / 2];                 // tile kt, group q, register r: element 4 (kt * NQ + q) + r
    __device__ __forceinline__ float get(int kt, int q, int r) const { const int i = 4 * (kt * S::NQ + q) + r; return v[i >> 4][i & 15]; }
    __device__ __forceinline__ void set(int kt, int q, int r, float x) { const int i = 4 * (kt * S::NQ + q) + r; v[i >> 4][i & 15] = x; }
};
// P^T of one step: words 0, 1 from tile 0, words 2, 3 from tile 1
template <class S>
struct Probs {
    u32x4 q[S::NQ];
};

// The accumulators as one value each at this point of the program.
template <class S, int D>
__device__ __forceinline__ void stream_pin(StreamRegs<S, D>& x)
{
#pragma unroll
    for (int b = 0; b < S::DT * S::NQ / 4; ++b) asm volatile("" : "+v"(x.acc[b]));
#pragma unroll
    for (int q = 0; q < S::NQ; ++q) asm volatile("" : "+v"(x.ls[q]));
}

// The probabilities exp2(c * s - m) of half HF of a step, spread over its MFMAs.  Pair k = query group
// k / 2, registers 2 (k % 2) .. + 1 of tile HF, in four parts: EXPONENTS, FIRST and SECOND exponential, PACK.
enum { EXPONENTS, FIRST, SECOND, PACK };
template <class S, int D, int HF, int K, int PART>
__device__ __forceinline__ void soft_part(StreamRegs<S, D>& x, const Scores<S>& st, float c, Probs<S>& p)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    constexpr int q = K / 2, r = 2 * (K % 2);
    if constexpr (PART == EXPONENTS) {
        x.x0 = __builtin_fmaf(st.get(HF, q, r), c, -x.m[q]);
        x.x1 = __builtin_fmaf(st.get(HF, q, r + 1), c, -x.m[q]);
        asm volatile("" : "+v"(x.x0), "+v"(x.x1));
    } else if constexpr (PART == FIRST) {
        x.e0 = __builtin_amdgcn_exp2f(x.x0);
        asm volatile("" : "+v"(x.e0));
    } else if constexpr (PART == SECOND) {
        x.e1 = __builtin_amdgcn_exp2f(x.x1);
        asm volatile("" : "+v"(x.e1));
    } else {
        bf16x2 pr;
        pr[0] = (__bf16)x.e0;
        pr[1] = (__bf16)x.e1;
        unsigned w = __builtin_bit_cast(unsigned, pr);
        if constexpr (K % 2 == 1) {
            x.seen = x.seen | p.q[q][2 * HF] | w;
            asm volatile("" : "+v"(w), "+v"(x.seen));
        } else asm volatile("" : "+v"(w));
        p.q[q][2 * HF + K % 2] = w;
    }
}

// What goes beside MFMA U of the half.  The parts beside one MFMA do not depend on each other.
template <class S, int D, int HF, int U>
__device__ __forceinline__ void soft_unit(StreamRegs<S, D>& x, const Scores<S>& st, float c, Probs<S>& p)
{
    if constexpr (S::UPM == 1) {
        soft_part<S, D, HF, U / 4, U % 4>(x, st, c, p);
    } else {
        constexpr int k = U / 2;
        if constexpr (U % 2 == 0) {
            if constexpr (k > 0) soft_part<S, D, HF, k - 1, PACK>(x, st, c, p);
            soft_part<S, D, HF, k, EXPONENTS>(x, st, c, p);
        } else {
            soft_part<S, D, HF, k, FIRST>(x, st, c, p);
            soft_part<S, D, HF, k, SECOND>(x, st, c, p);
            if constexpr (k == S::HALF - 1) soft_part<S, D, HF, k, PACK>(x, st, c, p);
        }
    }
}

template <class S, int D, int HF, int U = 0>
__device__ __forceinline__ void soft_half(StreamRegs<S, D>& x, const Scores<S>& st, float c, Probs<S>& p)
{
    if constexpr (U < S::UNITS) {
        soft_unit<S, D, HF, U>(x, st, c, p);
        soft_half<S, D, HF, U + 1>(x, st, c, p);
    }
}

// Largest exponent of a query of group q over the step (-inf where none of its keys is valid).
template <class S>
__device__ __forceinline__ float step_max(const Scores<S>& st, int q, float c)
{
    float mx = st.get(0, q, 0);
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, st.get(kt, q, r));
    // swaps of rows 1, 3 with rows 0, 2, then of the upper with the lower half: pairwise maxima
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1])) * c;
}

// Range of the exponents.  The reference m of a query is the maximum of its first step plus UP (of the stream: 16 unless said
// otherwise), so that probabilities of 2 and more mean a later maximum more than UP + 1 above the first.  Such a value has the
// top bit of its bf16 exponent set, which the or over all packed words shows; only then the references of that group of
// queries move up to the step's maximum (plus UP_AGAIN, 24), the sums and the accumulators are rescaled and the step's
// probabilities are made again.  What lies 2^(126 - UP) below a row's first maximum (2^(126 - UP_AGAIN) below a later one) is
// lost.
// How far up: the accumulators hold V times these weights, at most 2^-16 in an ordinary row, so V of 2^-110 is summed
// in normal numbers and smaller ones in subnormals with the precision of bf16 down to 2^-122 (with 60 in its place
// everything below 2^-89 came out as 0); each step less makes peaked rows move more often.  us, dense, D = 128 (1, 24,
// 4608) / D = 64 (2, 24, 4480), scores of standard deviation 1, 4, 16: 60 and 60 up 211 214 213 / 227 228 230; 8 and 8,
// all groups moved at once 212 228 272 / 226 256 344; 16 and 24 212 217 242 / 228 234 271; the 32x32x16 kernels before
// 235 245 253 / 269 274 275.  A test for 2^8 that needs no offset (a maximum over the packed words,
// v_pk_maximum3_f16, in place of the or) costs every dense call 1.5 %.
// 64-token masks take 4 and 4: values of V keep bf16's precision down to 2^-120 where scores climb (16 and 24: 2^-114), and
// the largest weight of a peaked row, which is exact where it is a reference, is one more often.  Error against 64 bits
// (10^-3 of the norm), H = 24, N = 2816, all ones, D = 128, scores of standard deviation 1, 2, 4, 8, 16: 32x32x16 kernel before
// 2.328 2.196 1.857 1.700 1.497 at 223 224 234 252 263 us; 16 and 24 2.332 2.212 1.913 1.749 1.527 at 122 122 123 129 140;
// 8 and 8 2.332 2.204 1.868 1.713 1.507 at 122 122 132 146 155; 4 and 4 2.331 2.093 1.812 1.691 1.499 at 121 130 143 154 159.

// Whether group q is among those.
template <class S>
__device__ __forceinline__ bool group_out(const Probs<S>& p, int q)
{
    const unsigned w = p.q[q][0] | p.q[q][1] | p.q[q][2] | p.q[q][3];
    return __builtin_amdgcn_ballot_w64((w & 0x40004000u) != 0u) != 0ull;
}
// The step's probabilities of those groups again.
template <class S, int D, int Q = 0, int I = 0>
__device__ __forceinline__ void soft_group(StreamRegs<S, D>& x, const Scores<S>& st, float c, Probs<S>& p)
{
    if constexpr (I < 16) {
        soft_part<S, D, I / 8, 2 * Q + I / 4 % 2, I % 4>(x, st, c, p);
        soft_group<S, D, Q, I + 1>(x, st, c, p);
    }
}
template <class S, int D, int Q = 0>
__device__ __forceinline__ void soft_groups(StreamRegs<S, D>& x, const Scores<S>& st, float c, Probs<S>& p)
{
    if constexpr (Q < S::NQ) {
        if (group_out<S>(p, Q)) soft_group<S, D, Q>(x, st, c, p);
        soft_groups<S, D, Q + 1>(x, st, c, p);
    }
}
template <class S, int D>
__device__ __forceinline__ void soft_close(StreamRegs<S, D>& x, const Scores<S>& st, float c, Probs<S>& p)
{
    unsigned long long out = __builtin_amdgcn_ballot_w64((x.seen & 0x40004000u) != 0u);
    if (__builtin_expect(out != 0ull, 0)) {
#pragma unroll
        for (int q = 0; q < S::NQ; ++q) {
            float alpha = 1.f;
            if (group_out<S>(p, q)) {
                const float m = fmaxf(x.m[q], step_max<S>(st, q, c) + S::UP_AGAIN);
                alpha = __builtin_amdgcn_exp2f(x.m[q] - m);
                x.m[q] = m;
            }
            asm volatile("" : "+v"(x.m[q]), "+v"(alpha));
            x.ls[q] *= alpha;
#pragma unroll
            for (int b = 0; b < S::DT; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) x.acc[(b * S::NQ + q) >> 2][((b * S::NQ + q) & 3) * 4 + r] *= alpha;
        }
        stream_pin<S, D>(x);                      // in place, before anything else is made
        asm volatile("" : "+s"(out));
    }
    if (__builtin_expect(out != 0ull, 0)) {       // (in a block of its own: together they need a second set of accumulators)
        soft_groups<S, D>(x, st, c, p);
        x.seen = 0u;
    }
}

// Keys at or beyond kv_len -> -inf, for a step whose first key is key0.
template <class S>
__device__ __forceinline__ void mask_step(Scores<S>& st, int key0, int kv_len, int lane)
{
    if (__builtin_expect(key0 + 32 > kv_len, 0)) {
        const int left = kv_len - key0 - 4 * (lane >> 4);
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int q = 0; q < S::NQ; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = st.get(kt, q, r);
                    st.set(kt, q, r, 16 * kt + r >= left ? -INFINITY : v);
                }
    }
}

// MFMAs of score item J
template <class S, int D, int J, int Q>
__device__ __forceinline__ void qk_mfma(StreamRegs<S, D>& x, Scores<S>& sn)
{
    constexpr int t = J / 2, kt = J % 2;
    constexpr int at = kt * S::NQ + Q;
    mfma16<at & 3>(sn.v[at >> 2], __builtin_bit_cast(bf16x8, x.kf[J % S::NBUF]), x.qf[Q][t], t == 0);
}
// MFMAs of output item J (counted from NQK); the row sums ride on the first NQ of them
template <class S, int D, int J, int Q>
__device__ __forceinline__ void pv_mfma(StreamRegs<S, D>& x, const Probs<S>& p)
{
    constexpr int slot = (J + S::NQK) % S::NBUF;
    const u32x4 both = __builtin_shufflevector(x.lo[slot], x.hi[slot], 0, 1, 2, 3);
    const bf16x8 pq = __builtin_bit_cast(bf16x8, p.q[Q]);
    constexpr int at = J * S::NQ + Q;
    mfma16<at & 3>(x.acc[at >> 2], __builtin_bit_cast(bf16x8, both), pq);
    if constexpr (J == Q) x.ls[Q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.ones, pq, x.ls[Q], 0, 0, 0);
}

// MFMAs Q .. NQ-1 of item I, each followed by its softmax units.  Every other item takes its query groups backwards, so
// that neighbouring MFMAs share one operand across the items too: less toggles on the way in, and the clock of a full chip
// is a matter of power (dense D = 128, N = 16896 2641 -> 2614 us; 0.3 to 0.6 % on every other kernel of the stream).
// Item I has arrived; after the first MFMA the wait for item I + 1 (not right before its use: the compiler would pad that).
template <class S, int D, bool QK, int I, int Q, int LAST, class Soft>
__device__ __forceinline__ void item_body(StreamRegs<S, D>& x, Scores<S>& sn, const Probs<S>& p, Soft soft)
{
    if constexpr (Q < S::NQ) {
        constexpr int J = QK ? I : I - S::NQK;
        constexpr int G = J % 2 ? S::NQ - 1 - Q : Q;
        if constexpr (QK) qk_mfma<S, D, J, G>(x, sn);
        else pv_mfma<S, D, J, G>(x, p);
        __builtin_amdgcn_sched_barrier(0);
        soft(std::integral_constant<int, J * S::NQ + Q>());
        if constexpr (Q == 0 && I + 1 < LAST) stream_wait<S, D, I + 1, LAST>(x);
        __builtin_amdgcn_sched_barrier(0);
        item_body<S, D, QK, I, Q + 1, LAST>(x, sn, p, soft);
    }
}

// First half of a step: S_{i+1} beside the second half of step i's probabilities.
template <class S, int D, int KC, int KN, int VC, int I, class Hook>
__device__ __forceinline__ void step_qk(StreamRegs<S, D>& x, const Scores<S>& sc, Scores<S>& sn, float c, Probs<S>& p, Hook hook)
{
    if constexpr (I < S::NQK) {
        stream_request<S, D, KC, KN, VC, I + S::PD>(x);
        item_body<S, D, true, I, 0, I + S::PD + 1>(x, sn, p, [&](auto u) {
            soft_unit<S, D, 1, decltype(u)::value>(x, sc, c, p);
        });
        hook(std::integral_constant<int, I>());
        step_qk<S, D, KC, KN, VC, I + 1>(x, sc, sn, c, p, hook);
    }
}

// Second half: O beside the first half of step i+1's probabilities.
template <class S, int D, int KC, int KN, int VC, int I, class Hook>
__device__ __forceinline__ void step_pv(StreamRegs<S, D>& x, Scores<S>& sn, float c, const Probs<S>& p, Probs<S>& pn, Hook hook)
{
    if constexpr (I < S::NI) {
        stream_request<S, D, KC, KN, VC, I + S::PD>(x);
        item_body<S, D, false, I, 0, I + S::PD + 1>(x, sn, p, [&](auto u) {
            soft_unit<S, D, 0, decltype(u)::value>(x, sn, c, pn);
        });
        hook(std::integral_constant<int, I>());
        step_pv<S, D, KC, KN, VC, I + 1>(x, sn, c, p, pn, hook);
    }
}

// The last step has no successor: its PV items alone.
template <class S, int D, int I, bool REQUEST_ONLY>
__device__ __forceinline__ void last_pv(StreamRegs<S, D>& x, const Probs<S>& p)
{
    if constexpr (REQUEST_ONLY) {
        if constexpr (I < S::NQK + S::PD) {
            stream_request<S, D, 0, 0, 0, I>(x);
            last_pv<S, D, I + 1, true>(x, p);
        }
    } else if constexpr (I < S::NI) {
        if constexpr (I + S::PD < S::NI) stream_request<S, D, 0, 0, 0, I + S::PD>(x);
        if constexpr (I == S::NQK) stream_wait<S, D, I, (I + S::PD < S::NI ? I + S::PD + 1 : S::NI)>(x);
        Scores<S> none;
        item_body<S, D, false, I, 0, (I + S::PD < S::NI ? I + S::PD + 1 : S::NI)>(x, none, p, [](auto) {});
        last_pv<S, D, I + 1, false>(x, p);
    }
}

// The scores of one step on their own: request the first PD items (REQUEST_ONLY), then run them.
template <class S, int D, int KC, int I, bool REQUEST_ONLY>
__device__ __forceinline__ void first_qk(StreamRegs<S, D>& x, Scores<S>& sn)
{
    if constexpr (REQUEST_ONLY) {
        if constexpr (I < S::PD && I < S::NQK) {
            stream_request<S, D, KC, KC, 0, I>(x);
            first_qk<S, D, KC, I + 1, true>(x, sn);
        }
    } else if constexpr (I < S::NQK) {
        if constexpr (I + S::PD < S::NQK) stream_request<S, D, KC, KC, 0, I + S::PD>(x);
        if constexpr (I == 0) stream_wait<S, D, 0, (S::PD < S::NQK ? S::PD + 1 : S::NQK)>(x);
        Probs<S> none;
        item_body<S, D, true, I, 0, (I + S::PD < S::NQK ? I + S::PD + 1 : S::NQK)>(x, sn, none, [](auto) {});
        first_qk<S, D, KC, I + 1, false>(x, sn);
    }
}

// Byte offset of this lane's chunk in its row, in a copy instruction (1 KB of the stage) whose row of this lane is `row`.
template <class S, int D, bool IS_V>
__device__ __forceinline__ unsigned stream_copy_chunk(int row, int lane)
{
    typedef Geo<D> G;
    return (unsigned)((lane % G::CPR) ^ (IS_V ? S::swz_v(row) : S::swz_k(row))) * 16u;
}

// Q^T operands requested by explicit assembly (see load_q_async): lane (n, g) holds elements
// 32 t + 8 g .. + 7 of query 16 q + n.  Rows at or beyond kv_len lie outside the buffer and come as zeros.
template <class S, int D>
__device__ __forceinline__ void stream_load_q(const Rows& Q, int q0, int kv_len, int lane, u32x4 (&raw)[S::NQ][S::KS])
{
    const TileBuffer b = tile_buffer<16 * S::NQ>(Q, q0, kv_len);
    const i32x4 rsrc = {(int)b.lo, (int)b.hi, (int)b.bytes, 0x00020000};
    const unsigned off = (unsigned)(lane & 15) * Q.row_bytes + (unsigned)(lane >> 4) * 16u;
#pragma unroll
    for (int q = 0; q < S::NQ; ++q)
#pragma unroll
        for (int t = 0; t < S::KS; ++t) {
            const unsigned at = off + (unsigned)(16 * q) * Q.row_bytes;
            // (five wait states behind a vector instruction that wrote the descriptor, which the compiler does not see to here)
            if (q == 0 && t == 0) asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %0, %1, %2, 0 offen" : "=v"(raw[q][t]) : "v"(at), "s"(rsrc));
            else asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen offset:%3" : "=v"(raw[q][t]) : "v"(at), "s"(rsrc), "i"(64 * t));
        }
}
template <class S, int D>
__device__ __forceinline__ void stream_q_arrived(StreamRegs<S, D>& x, u32x4 (&raw)[S::NQ][S::KS])
{
#pragma unroll
    for (int q = 0; q < S::NQ; ++q)
#pragma unroll
        for (int t = 0; t < S::KS; ++t) {
            asm volatile("" : "+v"(raw[q][t]));
            x.qf[q][t] = __builtin_bit_cast(bf16x8, raw[q][t]);
        }
}

// O = acc / l as bf16, query rows q0 .. q0 + 16 NQ - 1 of this wavefront; rows at or beyond kv_len and
// rows without any kept key become 0.  Through LDS (`stage`, 16 NQ rows of D * 2 + 16 bytes that nobody
// else uses) so that a store instruction covers whole rows: a lane holds 8-byte pieces of NQ rows.
// Bound by instruction issue (3700 cycles of a workgroup that shares its SIMDs with another, D = 128, 32 queries a wavefront), and
// nothing of it overlaps with products of the same workgroup, so a row that is zero is not chosen element by element but
// written over in LDS, where there is one, and the rows (all in one segment: 16 NQ divides 128) are one scalar base and
// 32-bit offsets.  us, rows of n kept blocks, before / now: D = 128, 64-token masks, N = 2048, H = 64, n = 4 48.6 / 46.5, 24 120.1 /
// 116.9; 128-token masks, N = 4096, n = 4 83.9 / 82.0, 24 342.7 / 340.8; D = 64, H = 256, n = 4 192.3 / 189.4.
// The columns of blocks B0 .. B1 - 1 of a row alone take RS = (B1 - B0) * 32 + 16 bytes of the stage.
template <class S, int D, int B0 = 0, int B1 = S::DT>
__device__ __forceinline__ void stream_output_rows(const StreamRegs<S, D>& x, const Rows& O, int q0, int kv_len, int N, int lane,
                                                   char* stage)
{
    constexpr int RS = (B1 - B0) * 32 + 16;
    const int n = lane & 15, g = lane >> 4;
    const u32x2 none = {0u, 0u};
#pragma unroll
    for (int q = 0; q < S::NQ; ++q) {
        const float l = x.ls[q][0];
        const float inv = 1.0f / l;
        const bool valid = q0 + 16 * q + n < kv_len && l > 0.f && inv != 0.f;
        char* const at = stage + (16 * q + n) * RS + 8 * g;
#pragma unroll
        for (int b = B0; b < B1; ++b) {
            bf16x4 ov;
#pragma unroll
            for (int r = 0; r < 4; ++r) ov[r] = (__bf16)(x.acc[(b * S::NQ + q) >> 2][((b * S::NQ + q) & 3) * 4 + r] * inv);
            *(bf16x4*)(at + 32 * (b - B0)) = ov;
        }
        if (__builtin_amdgcn_ballot_w64(!valid) != 0ull) {
            if (!valid) {
#pragma unroll
                for (int b = B0; b < B1; ++b) *(u32x2*)(at + 32 * (b - B0)) = none;
            }
        }
    }
    constexpr int CH = (B1 - B0) * 2;             // 16-byte chunks of a row
    constexpr int RPI = 64 / CH;                  // rows per store instruction
    const int rr = lane / CH, cc = lane % CH;
    char* const base = const_cast<char*>(O.row(q0)) + B0 * 32;
    const unsigned off = (unsigned)rr * O.row_bytes + (unsigned)cc * 16u;
    auto store = [&](auto all) {
#pragma unroll
        for (int i = 0; i < 16 * S::NQ / RPI; ++i) {
            const u32x4 v = *(const u32x4*)(stage + (i * RPI + rr) * RS + cc * 16);
            if (decltype(all)::value || q0 + i * RPI + rr < N) *(u32x4*)(base + (off + (unsigned)(i * RPI) * O.row_bytes)) = v;
        }
    };
    if (q0 + 16 * S::NQ <= N) store(std::true_type());
    else store(std::false_type());
}

// step(U), step(U + 1), .. at i + U, i + U + 1, ..
template <int U, int TO, class Step>
__device__ __forceinline__ void static_steps(Step& step, int i)
{
    if constexpr (U < TO) {
        step(std::integral_constant<int, U>(), i + U);
        static_steps<U + 1, TO>(step, i);
    }
}
// The same until step last - 1 has run: then end(U + 1) and true.
template <int U, int TO, class Step, class End>
__device__ __forceinline__ bool static_steps_until(Step& step, End& end, int i, int last)
{
    if constexpr (U < TO) {
        step(std::integral_constant<int, U>(), i + U);
        if (i + U + 1 == last) {
            end(std::integral_constant<int, U + 1>());
            return true;
        }
        return static_steps_until<U + 1, TO>(step, end, i, last);
    } else {
        return false;
    }
}

// ---------------------------------------------------------------------------
// The stream over a list of key tiles.  WQ x WK wavefronts: query group wq = wave / WK owns 16 NQ queries, key
// group wk = wave % WK the wk-th 32 keys of every 32 WK; with WK > 1 the key groups keep softmax states of
// their own and are merged at the end.  A tile = SPT steps of all key groups = 32 WK SPT keys, copied by
// all wavefronts into a ring of NSK stages for K and one of NSV stages for V.
//
// One barrier per tile, in the middle of the tile's first step (after S_{i+1}, before O).  At the barrier of
// tile t every wavefront has read K up to the rows of S_{i+1} and V_{t-1}, and has waited for its share of
// the next tiles' copies, so after it
//   SPT = 1: K_{t+2}, V_{t+1} may be read; the stages of K_{t+1}, V_{t-1} take K_{t+1+NSK}, V_{t-1+NSV}
//   SPT = 2: K_{t+1}, V_{t+1} may be read; the stages of K_t,     V_{t-1} take K_{t+NSK},   V_{t-1+NSV}
// Copies are issued V before K at every barrier and complete in order, which gives the counts below.
// ---------------------------------------------------------------------------
template <int D_, int NQ_, int WQ_, int WK_, int SPT_, int NSK_, int NSV_, int UP = 16, int UP_AGAIN = 24>
struct StreamPlan {
    static constexpr int D = D_, NQ = NQ_, WQ = WQ_, WK = WK_, SPT = SPT_, NSK = NSK_, NSV = NSV_;
    typedef Stream<D, NQ, 3, 4, UP, UP_AGAIN> S;
    static constexpr int NW = WQ * WK, QT = 16 * NQ * WQ, KTS = 32 * WK * SPT;
    static constexpr int TILE = KTS * S::RB;
    static constexpr int LC = TILE / 1024 / NW;   // copy instructions per wavefront per tile (K or V)
    static constexpr int LDS = (NSK + NSV) * TILE;
    static constexpr int gcd(int a, int b) { return b == 0 ? a : gcd(b, a % b); }
    static constexpr int UNROLL = NSK / gcd(NSK, NSV) * NSV * SPT;    // steps after which both rings are back at stage 0
    // Copies behind one write of M0.  Two: dense D = 64 0.5 to 3 % (most where items are cut), others up to 0.3 %; in the
    // short rings of the small kernel they are 0.5 (D = 64) to 2.5 % slower than copies spread out singly.
    static constexpr int PER_M0 = NSK >= 4 ? 2 : 1;
    static_assert(LC % PER_M0 == 0 && LC * NW * 1024 == TILE && (WK == 1 || SPT == 1) && NSK >= 2 && NSV >= 3, "");
    static constexpr int KLEAD = SPT == 1 ? NSK + 1 : NSK, VLEAD = NSV - 1;    // tiles ahead of t that are copied at its barrier
    // copy instructions that may still be on their way at a barrier
    static constexpr int min(int a, int b) { return a < b ? a : b; }
    static constexpr int LOOSE = min(LC + 2 * LC * (NSV - 3), 2 * LC * (NSK - 2));
    // byte offset of the 32 rows of step i (of key group 0) in the K and the V ring
    static constexpr __host__ __device__ int k_off(int i) { return (i / SPT % NSK) * TILE + (i % SPT) * 32 * S::RB; }
    static constexpr __host__ __device__ int v_off(int i) { return (i / SPT % NSV) * TILE + (i % SPT) * 32 * S::RB; }
};

// Where a run ends, as Keys::LAST: the number of its last step modulo UNROLL where that is known when compiling; ANY: what is left
// over after whole runs of the unrolled loop goes through a second copy of it that can be left after every step; SHORT: so few
// steps that the loop itself can be.  (Steps outside the unrolled loop added up LDS addresses, moved the scores and issued their copies
// all at once.)  us, such steps / now: SHORT, rows of 2, 4, 24 64-token blocks, D = 128, H = 64, N = 2048 39.9 48.7 120.8 / 37.5 44.0
// 113.9; ANY, dense, D = 128, N = 4608 (7 of 143 steps) 216.3 / 213.3, D = 64, B = 2, N = 4480 226.5 / 224.5.  SHORT for dense calls:
// 0.4 to 1 % slower there, N = 16896, D = 128 0.5 %.
enum { ANY = -1, SHORT = -2 };
// Which tiles: at(t, ahead) is the first key of tile t; the caller stands in tile t - ahead and calls next_tile when it has
// done with a tile.  BLOCKS (KeptKeys): the same of whole blocks of four tiles, of which two, b0 and b1, are known.
// Tiles in order: the dense path.
template <class P>
struct AllKeys {
    static constexpr int LAST = ANY;
    static constexpr bool BLOCKS = false;
    __device__ __forceinline__ int at(int t, int) const { return t * P::KTS; }
    __device__ __forceinline__ void next_tile() {}
};

// The kept blocks of a row (or of a piece of one), in order.  Up to 64 blocks per side they are the bits of one scalar:
// from the row of the mask itself (a byte per lane, one ballot) or, where selection wrote lists, from the list; nothing in
// the loop then waits for memory.  Beyond, they come from the list, the next entry under way (128-token masks: a block is
// four steps) or 64 at a time, one per lane of `first` (a scalar load shares its counter with the LDS reads in flight, and
// a 64-key block is one step).  Past the end: NOWHERE, beyond every kv_len.
template <int BLOCK>
struct KeptBlocks {
    static constexpr int NOWHERE = 1 << 23;        // times 128 keys
    typedef const __attribute__((address_space(4))) int32_t* cptr_t;
    unsigned long long bits;
    const int32_t* list;                           // null: the bits
    int n, at, first;
    __device__ __forceinline__ void load()
    {
        if (BLOCK == 128) { first = ((cptr_t)list)[at < n ? at : 0]; return; }
        const int i = at + (int)(threadIdx.x & 63u);
        asm volatile("global_load_dword %0, %1, %2\n\ts_waitcnt vmcnt(0)" : "=&v"(first) : "v"((i < n ? i : 0) * 4), "s"(list) : "memory");
        first = i < n ? first : NOWHERE;
    }
    // The list out of line: 0.5 to 1 % for rows of up to 64 blocks on the streams, but 1 % against longer ones on the kernel of four
    // wavefronts per SIMD (us, D = 64, 132 blocks, density 0.2, out of line / not: H = 2 88.2 / 87.3, 4 103.7 / 102.4, 8 171.5 / 170.0).
    template <bool OUT_OF_LINE = true>
    __device__ __forceinline__ int next()
    {
        if (OUT_OF_LINE ? __builtin_expect(list == nullptr, 1) : list == nullptr) {
            const int j = bits != 0ull ? __builtin_ctzll(bits) : NOWHERE;
            bits &= bits - 1ull;
            return j;
        }
        if (BLOCK == 128) {
            const int j = at < n ? first : NOWHERE;
            ++at;
            load();
            return j;
        }
        if ((at & 63) == 0) load();
        return __builtin_amdgcn_readlane(first, at++ & 63);
    }
};

// What workgroup wg does: an entry of the plan (PLAN_READ); the entry that a plan of whole rows would have, which it finds by itself
// (PLAN_FOUND: find_row); or, where all rows are on the chip at once and none is long enough to be cut, so that their order says
// little, a row of its segment by its own number (PLAN_NONE).
// Where there is no plan to read, and for the lists wherever the rows come from the mask, it also leaves in the workspace what
// the planner kernels would have left there.
template <int BLOCK>
struct SparseWork {
    PlanRec rec;
    KeptBlocks<BLOCK> kept;
    unsigned long long row;                        // all kept blocks of the row, where they come from the mask
};
// Its entry: the dispatcher deals workgroups out to the 8 XCDs in turn, so segment x = wg % 8 is XCD x's.  Fewer (sample,
// head) pairs than XCDs (a rank of a model whose heads are dealt out over ranks) would leave XCDs idle: from 24 rows per pair
// on the workgroups are dealt out to the segments that hold items, each of which then runs on its share of the chip.  The
// K/V of a head are in several L2s then, which pays least where little is kept of many keys and pairs and XCDs do not
// divide, so not for 5 to 7 pairs under 64-token masks.  us, one XCD per pair / spread, densities 0.1 0.3 0.8:
//   128-token masks, D = 128, H = 1, N = 16896 127 297 746 / 63 123 275; 2, 8192 57 104 211 / 42 63 126; B = 2, H = 2,
//     N = 16896 147 350 894 / 92 211 547; 3, 2, 4480 41 48 90 / 37 45 86; D = 64, 1, 2, 16896 94 219 537 / 58 112 247
//   64-token masks, D = 128, 1, 2, 16896 186 357 875 / 177 186 313; 2, 2, 3840 47 51 61 / 39 40 40; the slowest of 1 to 4
//     pairs 1, 3, 16896 186 359 874 / 191 199 377, of 6 pairs 3, 2, 16896 191 369 899 / 225 349 712
//   few rows: D = 128, 1, 2, 1024 (8 rows per pair) 20.8 / 21.2, 2048 30.6 30.9 39.8 / 31.1 31.0 40.4
// The segments without items come last.
__device__ __forceinline__ void entry_of(const AttnParams& p, int& seg, int& i)
{
    const unsigned wg = blockIdx.x;
    seg = wg % XCDS;
    i = wg / XCDS;
    if (p.segs < XCDS) {                           // the same for the whole launch
        // (the quotient is exact below 2^32 / segs; segs = 1: the magic number wraps to 0)
        i = p.segs == 1 ? wg : __umulhi(wg, p.seg_magic);
        seg = wg - i * p.segs;
        if (i >= p.chunk) {
            const int over = wg - p.segs * p.chunk;
            seg = __builtin_amdgcn_readfirstlane(p.segs + over / p.chunk);    // (a division is vector instructions)
            i = __builtin_amdgcn_readfirstlane(over % p.chunk);
        }
    }
}
// The entry of a plan of whole rows that nobody has made: every workgroup counts all rows of its segment, one per
// thread (8 <= nb <= 64), and looks up the one that comes i-th, longest first (with the second round of 32 backwards, FOURTH:
// the fourth too: see plan_small_kernel).  `at`: LDS that no copy uses yet.
// Some 1.5 us of every workgroup in place of a launch: run_sparse holds both sides of the line.
constexpr int FOUND_ROWS = 256;                  // rows of a segment, at most: the threads of a workgroup
struct FoundRow {
    int hist[SMALL_NB + 2];                        // rows by length, longest first
    int before[FOUND_ROWS / 64];                   // rows of the length looked for, by 64 rows
    int item, n;
    unsigned long long row;
};
template <int BLOCK, bool FOURTH>
__device__ __forceinline__ void find_row(const AttnParams& p, int seg, int i, SparseWork<BLOCK>& w, FoundRow* at)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nb = p.nb;
    const int items = (p.pairs - seg + XCDS - 1) / XCDS * nb;
    if (i >= items) return;
    const bool has = tid < items;
    const int t = has ? tid : 0;
    const int pair = (int)__umulhi((unsigned)t, p.nq.magic) * XCDS + seg;    // (nq = nb)
    const int item = pair * nb + t - (pair - seg) / XCDS * nb;
    int c;
    unsigned long long row = 0ull;
    if (p.mask != nullptr) {
        int kv_len = p.kv_len;
        if (p.kv_lens != nullptr) kv_len = p.kv_lens[p.H.d == 1 ? pair : (int)__umulhi((unsigned)pair, p.H.magic)];
        kv_len = kv_len < 0 ? 0 : (kv_len > p.N ? p.N : kv_len);
        const unsigned char* src = p.mask + (size_t)item * nb;
        unsigned long long v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)                // all on their way at once; the last eight bytes of a row end with it
            if (8 * k < nb) __builtin_memcpy(&v[k], src + (8 * k + 8 <= nb ? 8 * k : nb - 8), 8);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (8 * k < nb) row |= (unsigned long long)byte_bits((unsigned)v[k], (unsigned)(v[k] >> 32)) << (8 * k + 8 <= nb ? 8 * k : nb - 8);
        const int live = (kv_len + BLOCK - 1) / BLOCK;
        row &= live >= 64 ? ~0ull : (1ull << live) - 1ull;
        c = __popcll(row);
    } else {
        c = p.counts[item];
    }
    if (tid <= nb) at->hist[tid] = 0;
    __syncthreads();
    if (has) atomicAdd(&at->hist[nb - c], 1);
    __syncthreads();
    auto backwards = [&](int first) {              // a round of 32
        const int left = items - first < CUS_PER_XCD ? items - first : CUS_PER_XCD;
        if (i >= first && i < first + CUS_PER_XCD) i = first + left - 1 - (i - first);
    };
    backwards(CUS_PER_XCD);
    if (FOURTH) backwards(3 * CUS_PER_XCD);
    const int upto = wave_scan_inclusive(lane < nb ? at->hist[lane] : 0);
    const int shorter = __popcll(__builtin_amdgcn_ballot_w64(lane < nb && upto <= i));    // nb - the length of the i-th row
    const int start = shorter > 0 ? __builtin_amdgcn_readlane(upto, shorter - 1) : 0;
    const bool as_long = has && nb - c == shorter;
    const unsigned long long same = __builtin_amdgcn_ballot_w64(as_long);
    if (lane == 0) at->before[wave] = __popcll(same);
    __syncthreads();
    int rank = __popcll(same & ((1ull << lane) - 1ull));
#pragma unroll
    for (int k = 0; k < FOUND_ROWS / 64 - 1; ++k) rank += k < wave ? at->before[k] : 0;
    if (as_long && rank == i - start) { at->item = item; at->n = c; at->row = row; }
    __syncthreads();
    w.rec.item = __builtin_amdgcn_readfirstlane(at->item);
    w.rec.nblk = __builtin_amdgcn_readfirstlane(at->n);
    const unsigned long long r = at->row;
    w.row = (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(r >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((int)r);
}

// ROUNDS: of rows that are looked up, 2 or 4; 0: a kernel whose calls always have a plan (256 threads where not).
template <int BLOCK, int ROUNDS>
__device__ __forceinline__ SparseWork<BLOCK> sparse_work(const AttnParams& p, char* scratch)
{
    typedef const __attribute__((address_space(4))) int32_t* cptr_t;
    typedef const __attribute__((address_space(4))) i32x4* rptr_t;
    static_assert(sizeof(PlanRec) == sizeof(i32x4), "one record = one 16-byte scalar load");
    arguments_at_hand(p);
    int seg, i;
    entry_of(p, seg, i);
    const int slot = seg * p.chunk + i, lane = threadIdx.x & 63;
    SparseWork<BLOCK> w;
    w.rec = {-1, 0, 0, -1};
    w.row = 0ull;
    const int planned = ROUNDS > 0 ? p.planned : PLAN_READ;
    if (planned == PLAN_FOUND) {
        find_row<BLOCK, ROUNDS == 4>(p, seg, i, w, (FoundRow*)scratch);
    } else if (planned == PLAN_NONE) {
        // The dispatcher deals the workgroups of an XCD out to its 32 CUs in turn; rows with the same number (text rows,
        // the long ones) would meet on the same CU where 32 is a multiple of nb, so every 32 workgroups start 3/8 of the rows on.
        const int g = p.nq.of(i), pair = g * XCDS + seg;    // (nq = nb)
        if (pair * p.nb < p.items) {
            const int turned = i + g * p.nb / CUS_PER_XCD * ((3 * p.nb + 7) / 8);
            w.rec.item = pair * p.nb + turned - p.nq.of(turned) * p.nb;
            if (p.mask == nullptr) w.rec.nblk = ((cptr_t)p.counts)[w.rec.item];
        }
    } else if (BLOCK == 64) {
        w.rec.item = ((cptr_t)p.order)[slot];
        if (w.rec.item >= 0) w.rec.nblk = ((cptr_t)p.counts)[w.rec.item];
    } else {
        const i32x4 raw = ((rptr_t)p.order)[slot];
        w.rec = {raw[0], raw[1], raw[2], raw[3]};
    }
    const int item = w.rec.item;
    w.kept.list = nullptr;
    w.kept.bits = w.row;
    w.kept.n = w.rec.nblk;
    w.kept.at = w.kept.first = 0;
    if (item >= 0 && !(planned == PLAN_FOUND && p.mask != nullptr)) {
        if (p.mask != nullptr) {                   // nb <= 64
            int kv_len = p.kv_len;
            if (p.kv_lens != nullptr) kv_len = ((cptr_t)p.kv_lens)[p.H.of(p.nq.of(item))];    // (nq = nb)
            kv_len = kv_len > p.N ? p.N : kv_len;
            const unsigned char byte = p.mask[(size_t)item * p.nb + (lane < p.nb ? lane : 0)];
            const bool keep = byte != 0 && lane < p.nb && lane * BLOCK < kv_len;
            w.kept.bits = w.row = __builtin_amdgcn_ballot_w64(keep);
            if (planned == PLAN_NONE) {
                w.rec.nblk = __popcll(w.row);
            } else if (BLOCK == 128 && w.rec.w >= 0) {
                const int rank = __popcll(w.row & ((1ull << lane) - 1ull)) - w.rec.blk0;
                w.kept.bits = __builtin_amdgcn_ballot_w64(keep && rank >= 0 && rank < w.rec.nblk);
            }
        } else if (p.nb <= 64) {
            // every lane sends a 1 to the lane of its entry (lanes without one to that of the first)
            const int j = p.index[(size_t)item * p.nb + w.rec.blk0 + (lane < w.rec.nblk ? lane : 0)];
            const unsigned long long row = __builtin_amdgcn_ballot_w64(__builtin_amdgcn_ds_permute(4 * j, 1) != 0);
            w.kept.bits = w.rec.nblk > 0 ? row : 0ull;
        } else {
            w.kept.list = p.index + (size_t)item * p.nb + w.rec.blk0;
            if (BLOCK == 128 && w.rec.nblk > 0) w.kept.load();
        }
    }
    return w;
}

// The workspace as the planner kernels would have left it: called behind the loop, whose waits for copies would wait for
// these stores as well.
template <int BLOCK, int ROUNDS>
__device__ __forceinline__ void leave_plan(const AttnParams& p, const SparseWork<BLOCK>& w)
{
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x;
    if (p.mask != nullptr && (w.row >> lane & 1ull) != 0ull && w.rec.blk0 == 0)
        p.index[(size_t)w.rec.item * p.nb + __popcll(w.row & ((1ull << lane) - 1ull))] = lane;
    if (ROUNDS > 0 && p.planned != PLAN_READ && lane == 0) {
        int x, i;
        entry_of(p, x, i);
        if (BLOCK == 64) p.order[x * p.chunk + i] = w.rec.item;
        else ((PlanRec*)p.order)[x * p.chunk + i] = w.rec;
        // (counts that are there already are what other workgroups look their rows up by)
        if (p.mask != nullptr && w.rec.item >= 0) p.counts[w.rec.item] = w.rec.nblk;
        if (BLOCK == 128 && i < p.pmax) p.arrived[x * p.pmax + i] = 0;
    }
}

// The 32-key steps of kept 128-key blocks (four steps = one block = one run of the unrolled loop): first keys of the block
// under way and of the one after it.
template <class P>
struct KeptKeys {
    static_assert(P::KTS == 32 && P::UNROLL == 4 && P::KLEAD == 5 && P::VLEAD == 3, "");
    static constexpr int LAST = P::UNROLL - 1;
    static constexpr bool BLOCKS = true;
    KeptBlocks<128> kept;
    int b0, b1;
    __device__ __forceinline__ KeptKeys(const KeptBlocks<128>& kept_) : kept(kept_)
    {
        b0 = kept.next() * 128;
        b1 = kept.next() * 128;
    }
    __device__ __forceinline__ int at(int, int ahead) const { return ahead == 0 ? b0 : b1; }
    __device__ __forceinline__ void next_tile()
    {
        b0 = b1;
        b1 = kept.next() * 128;
    }
};

// Kept 64-key blocks, a block one tile: the first keys of the current tile and the three after it.
template <class P>
struct KeptTiles {
    static_assert(P::KTS == 64 && P::SPT == 1 && P::KLEAD == 3 && P::VLEAD == 2, "");
    static constexpr int LAST = SHORT;
    static constexpr bool BLOCKS = false;
    KeptBlocks<64> kept;
    int b0, b1, b2, b3;
    __device__ __forceinline__ KeptTiles(const KeptBlocks<64>& kept_) : kept(kept_)
    {
        b0 = kept.next() * 64;
        b1 = kept.next() * 64;
        b2 = kept.next() * 64;
        b3 = kept.next() * 64;
    }
    __device__ __forceinline__ int at(int, int ahead) const { return ahead == 0 ? b0 : ahead == 1 ? b1 : ahead == 2 ? b2 : b3; }
    __device__ __forceinline__ void next_tile()
    {
        b0 = b1;
        b1 = b2;
        b2 = b3;
        b3 = kept.next() * 64;
    }
};

// Steps 0 .. last of this workgroup's queries against the tiles of `keys` (tiles at or beyond kv_len are all masked).  The
// unrolled loop is left behind whichever of its steps is the last but one.
template <class P, class Keys>
__device__ __forceinline__ void stream_attend(StreamRegs<typename P::S, P::D>& x, char* lds, const Rows& Q, const Rows& K, const Rows& V,
                                              int q0, int kv_len, float c, int last, Keys& keys, int wave, int lane)
{
    typedef typename P::S S;
    constexpr int D = P::D, LC = P::LC;
    constexpr int VBASE = P::NSK * P::TILE;
    const int wk = wave % P::WK;
#pragma unroll
    for (int b = 0; b < S::DT * S::NQ / 4; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) x.acc[b][r] = 0.f;
#pragma unroll
    for (int q = 0; q < S::NQ; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) x.ls[q][r] = 0.f;

    u32x4 qraw[S::NQ][S::KS];
    stream_load_q<S, D>(Q, q0, kv_len, lane, qraw);
    unsigned koff[LC], voff[LC];
    const int copy_row = wave * LC * Geo<D>::ROWS_PER_LOAD + lane / Geo<D>::CPR;
    const unsigned copy_off = (unsigned)copy_row * K.row_bytes;    // (V's rows are as far apart)
#pragma unroll
    for (int e = 0; e < LC; ++e) {
        const int more = e * Geo<D>::ROWS_PER_LOAD;
        koff[e] = copy_off + (unsigned)more * K.row_bytes + stream_copy_chunk<S, D, false>(copy_row + more, lane);
        voff[e] = copy_off + (unsigned)more * K.row_bytes + stream_copy_chunk<S, D, true>(copy_row + more, lane);
    }
    const unsigned lds0 = (unsigned)(size_t)LDS_PTR(char, lds);
    unsigned dst0 = lds0 + (unsigned)(wave * LC) * 1024u;
    // (dst0 as it is here: else every stage's address is a register of its own, kept in lanes of a vector register)
    auto copy = [&](const TileBuffer& b, const unsigned (&off)[LC], int e, unsigned ahead) {
        asm volatile("" : "+s"(dst0));
        const unsigned dst = dst0 + ahead;
        if constexpr (P::PER_M0 == 1) copy_1k(b, off[e], dst);
        else if (e % 2 == 0) copy_2k(b, off[e], off[e + 1], dst);
    };
    auto copy_k = [&](const TileBuffer& b, int e, unsigned stage) { copy(b, koff, e, stage + e * 1024); };
    auto copy_v = [&](const TileBuffer& b, int e, unsigned stage) { copy(b, voff, e, VBASE + stage + e * 1024); };
    // Kept blocks: a descriptor is made for a whole block and moves on tile by tile, a third of the scalar instructions of one for
    // every tile.  us, one for every tile / now: H = 24, D = 128, N = 4608, densities 0.2 0.5 1 91.5 136.4 226.3 / 90.8 135.7 224.0; N = 1536
    // 33.2 / 32.5; D = 64, H = 256, N = 4096, 24 blocks a row 777 / 770.
    constexpr bool BLOCKS = Keys::BLOCKS;
    TileBuffer kb, vb;                            // the tiles being copied
    const unsigned tile_bytes = (unsigned)P::KTS * K.row_bytes;
    // what the barriers before tile 0 would have issued
    if constexpr (BLOCKS) {
        kb = tile_buffer<128>(K, keys.b0, kv_len);
        vb = tile_buffer<128>(V, keys.b0, kv_len);
#pragma unroll
        for (int b = -P::KLEAD; b < -1; ++b) {
            if (b >= -P::VLEAD) {
                if (b > -P::VLEAD) next_tile_of(vb, tile_bytes);
#pragma unroll
                for (int e = 0; e < LC; ++e) copy_v(vb, e, (b + P::VLEAD) * P::TILE);
            }
            if (b > -P::KLEAD) next_tile_of(kb, tile_bytes);
#pragma unroll
            for (int e = 0; e < LC; ++e) copy_k(kb, e, (b + P::KLEAD) * P::TILE);
        }
    } else
#pragma unroll
    for (int b = -P::KLEAD; b < (P::SPT == 1 ? -1 : 0); ++b) {
        if (b + P::VLEAD >= 0) {
            const TileBuffer vb = tile_buffer<P::KTS>(V, keys.at(b + P::VLEAD, b + P::VLEAD), kv_len);
#pragma unroll
            for (int e = 0; e < LC; ++e) copy_v(vb, e, (b + P::VLEAD) * P::TILE);
        }
        const TileBuffer kb = tile_buffer<P::KTS>(K, keys.at(b + P::KLEAD, b + P::KLEAD), kv_len);
#pragma unroll
        for (int e = 0; e < LC; ++e) copy_k(kb, e, (b + P::KLEAD) * P::TILE);
    }
    // copies issued so far that are younger than K_0 (SPT = 1), or than K_0 and V_0
    constexpr int ISSUED = P::SPT == 1 ? (P::NSK + (P::NSV - 2)) * LC : (P::NSK + P::NSV - 1) * LC;
    stream_addresses<S, D>(x, lds0 + wk * 32 * S::RB, lds0 + VBASE + wk * 32 * S::RB, lane);
    wait_vmcnt<ISSUED - (P::SPT == 1 ? LC : 2 * LC)>();
    stream_q_arrived<S, D>(x, qraw);
    const u32x4 one = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    x.ones = __builtin_bit_cast(bf16x8, one);
    asm volatile("" : "+v"(x.ones));              // kept in registers
    phase_barrier();

    Scores<S> st[2];
    Probs<S> pw;
    first_qk<S, D, 0, 0, true>(x, st[0]);
    first_qk<S, D, 0, 0, false>(x, st[0]);
    if constexpr (P::SPT == 1) {                  // the barrier before tile 0: K_1, V_0 may be read
        if constexpr (BLOCKS) {
            next_tile_of(vb, tile_bytes);
            kb = tile_buffer<128>(K, keys.b1, kv_len);
        } else {
            vb = tile_buffer<P::KTS>(V, keys.at(P::VLEAD - 1, P::VLEAD - 1), kv_len);
            kb = tile_buffer<P::KTS>(K, keys.at(P::KLEAD - 1, P::KLEAD - 1), kv_len);
        }
        wait_vmcnt<P::LOOSE>();
        phase_barrier();
#pragma unroll
        for (int e = 0; e < LC; ++e) copy_v(vb, e, (P::VLEAD - 1) * P::TILE);
#pragma unroll
        for (int e = 0; e < LC; ++e) copy_k(kb, e, 0);
    }
    mask_step<S>(st[0], keys.at(0, 0) + wk * 32, kv_len, lane);
#pragma unroll
    for (int q = 0; q < S::NQ; ++q) {
        x.m[q] = fmaxf(step_max<S>(st[0], q, c) + S::UP, REF_LOWEST);  // (a key group may have no valid key at all)
    }
    x.seen = 0u;
    soft_half<S, D, 0>(x, st[0], c, pw);

    // Step i.  U = i % UNROLL.
    auto step = [&](auto u, int i) {
        constexpr int U = decltype(u)::value;
        constexpr bool FIRST_OF_TILE = U % P::SPT == 0;
        Scores<S>& sc = st[U & 1];
        Scores<S>& sn = st[(U + 1) & 1];
        constexpr int KC = P::k_off(U + 1), KN = P::k_off(U + 2), VC = P::v_off(U);
        // the copies of this tile's barrier, one every few items until the next barrier (SPT = 1: in the
        // second half only)
        constexpr int SLOTS = P::SPT == 1 ? S::NPV : S::NPV + S::NI;
        constexpr int PER = (2 * LC + SLOTS - 1) / SLOTS, GAP = SLOTS / (2 * LC) > 0 ? SLOTS / (2 * LC) : 1;
        constexpr int T0 = U / P::SPT;
        auto hook = [&](auto item) {
            constexpr int at = decltype(item)::value - S::NQK + (U % P::SPT) * S::NI;
            if constexpr (at >= 0 && at % GAP == 0) {
#pragma unroll
                for (int e = at / GAP * PER; e < at / GAP * PER + PER && e < 2 * LC; ++e) {
                    if (e < LC) copy_v(vb, e, (T0 + P::VLEAD) % P::NSV * P::TILE);
                    else copy_k(kb, e - LC, (T0 + P::KLEAD) % P::NSK * P::TILE);
                }
            }
        };
        if constexpr (FIRST_OF_TILE) step_qk<S, D, KC, KN, VC, 0>(x, sc, sn, c, pw, [](auto) {});
        else step_qk<S, D, KC, KN, VC, 0>(x, sc, sn, c, pw, hook);
        soft_close<S, D>(x, sc, c, pw);
        const int t = i / P::SPT;
        mask_step<S>(sn, BLOCKS ? keys.at(0, U == 3 ? 1 : 0) + (U + 1) % 4 * 32
                         : P::SPT == 1 ? keys.at(t + 1, 1) + wk * 32 : keys.at((i + 1) / 2, 0) + (i + 1) % 2 * 32, kv_len, lane);
        if constexpr (FIRST_OF_TILE) {
            if constexpr (BLOCKS) {               // V_{t+3} and K_{t+5}
                if constexpr (U == 1) vb = tile_buffer<128>(V, keys.b1, kv_len);
                else next_tile_of(vb, tile_bytes);
                if constexpr (U == 3) {
                    keys.next_tile();
                    kb = tile_buffer<128>(K, keys.b1, kv_len);
                } else next_tile_of(kb, tile_bytes);
            } else {
                vb = tile_buffer<P::KTS>(V, keys.at(t + P::VLEAD, P::VLEAD), kv_len);
                kb = tile_buffer<P::KTS>(K, keys.at(t + P::KLEAD, P::KLEAD), kv_len);
                keys.next_tile();
            }
            wait_vmcnt<P::LOOSE>();
            phase_barrier();
        }
        Probs<S> pn;
        step_pv<S, D, KC, KN, VC, S::NQK>(x, sn, c, pw, pn, hook);
#pragma unroll
        for (int q = 0; q < S::NQ; ++q) { pw.q[q][0] = pn.q[q][0]; pw.q[q][1] = pn.q[q][1]; }
    };
    if (last > 0) {
        stream_pin<S, D>(x);
        first_qk<S, D, P::k_off(1), 0, true>(x, st[1]);     // the first items of step 0's stream
        stream_wait<S, D, 0, S::PD>(x);
        auto end = [&](auto u) { if constexpr (decltype(u)::value & 1) st[0] = st[1]; };
        int i = 0;
        if constexpr (Keys::LAST == SHORT) {
            for (;; i += P::UNROLL) {
                stream_pin<S, D>(x);
                if (static_steps_until<0, P::UNROLL>(step, end, i, last)) break;
            }
        } else {
            for (; i + P::UNROLL <= last; i += P::UNROLL) {
                stream_pin<S, D>(x);
                static_steps<0, P::UNROLL>(step, i);
            }
            if constexpr (Keys::LAST == ANY) {
                if (i < last) static_steps_until<0, P::UNROLL - 1>(step, end, i, last);
            } else {
                static_steps<0, Keys::LAST>(step, i);
                end(std::integral_constant<int, Keys::LAST>());
            }
        }
        stream_drain<S, D>(x);
    }
    soft_half<S, D, 1>(x, st[0], c, pw);
    soft_close<S, D>(x, st[0], c, pw);
#pragma unroll
    for (int b = 0; b < S::DT; ++b) x.vaddr[b] += P::v_off(last);
    last_pv<S, D, S::NQK, true>(x, pw);
    last_pv<S, D, S::NQK, false>(x, pw);
    wait_vmcnt<0>();                              // no copy may land once the stages serve something else
}

// The two key groups of a workgroup add their states up through LDS and store the result, each one half of the columns: it
// hands the other half of its accumulators over (with its references and sums), and the rows it stores go through what it has
// read of that.  (A group that saw no valid key has l = 0 and a reference far below every other.)  Every wavefront comes here,
// after a barrier that ends the use of the stages.  us, one group doing it all / now: rows of 2, 8, 16 64-token blocks,
// N = 2048, D = 128, H = 64 36.6 57.3 84.1 / 35.2 55.9 82.5; dense, in a graph, N = 256, H = 2, D = 128 5.40 / 5.18; 640, 24 11.6 / 11.1.
template <class P>
__device__ __forceinline__ void stream_merge_rows(StreamRegs<typename P::S, P::D>& x, char* lds, const Rows& O, int q0, int kv_len, int N,
                                                  int wave, int lane)
{
    typedef typename P::S S;
    constexpr int D = P::D, HALF = S::DT / 2;
    constexpr int GIVEN = 64 * (HALF * S::NQ * 16 + S::NQ * 8);    // bytes that a wavefront hands over
    static_assert(P::WK == 2 && P::NW * GIVEN <= P::LDS, "the states fit the stages");
    static_assert(16 * S::NQ * (HALF * 32 + 16) <= GIVEN, "and a wavefront's rows what it was given");
    const int wq = wave / 2;
    auto part = [&](auto group) {
        constexpr int WK = decltype(group)::value, KEEP = WK * HALF, GIVE = (1 - WK) * HALF;    // first blocks
        char* const mine = lds + (wq * 2 + WK) * GIVEN;             // what it is given
        char* const other = lds + (wq * 2 + 1 - WK) * GIVEN;
        auto quads = [&](char* at) { return (f32x4*)at + lane; };
        auto ml = [&](char* at) { return (float*)(at + 64 * HALF * S::NQ * 16) + lane * S::NQ * 2; };
#pragma unroll
        for (int i = 0; i < HALF * S::NQ; ++i) {
            f32x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = x.acc[(GIVE * S::NQ + i) >> 2][((GIVE * S::NQ + i) & 3) * 4 + r];
            quads(other)[i * 64] = v;
        }
#pragma unroll
        for (int q = 0; q < S::NQ; ++q) { ml(other)[2 * q] = x.m[q]; ml(other)[2 * q + 1] = x.ls[q][0]; }
        __syncthreads();
        float a[2][S::NQ];                        // factors of group 0's and of group 1's
        auto sum = [&](float kept, float given, int q) { return WK == 0 ? kept * a[0][q] + given * a[1][q] : given * a[0][q] + kept * a[1][q]; };
#pragma unroll
        for (int q = 0; q < S::NQ; ++q) {
            const float m1 = ml(mine)[2 * q], m = fmaxf(x.m[q], m1);
            a[WK][q] = __builtin_amdgcn_exp2f(x.m[q] - m);
            a[1 - WK][q] = __builtin_amdgcn_exp2f(m1 - m);
            x.ls[q][0] = sum(x.ls[q][0], ml(mine)[2 * q + 1], q);
        }
#pragma unroll
        for (int i = 0; i < HALF * S::NQ; ++i) {
            const f32x4 v = quads(mine)[i * 64];
            const int k = KEEP * S::NQ + i;
#pragma unroll
            for (int r = 0; r < 4; ++r) x.acc[k >> 2][(k & 3) * 4 + r] = sum(x.acc[k >> 2][(k & 3) * 4 + r], v[r], i % S::NQ);
        }
        stream_output_rows<S, D, KEEP, KEEP + HALF>(x, O, q0, kv_len, N, lane, mine);
    };
    if (wave % 2 == 0) part(std::integral_constant<int, 0>());
    else part(std::integral_constant<int, 1>());
}

// Dense plans.  D = 128: 8 wavefronts, 32 queries each, two per SIMD, 128 KB of LDS.  D = 64: 4 wavefronts of 64
// queries (32 in the quarters), 64 KB, two workgroups per CU.
template <int D> struct DensePlan {
    typedef StreamPlan<128, 2, 8, 1, 2, 4, 4> Whole;
    typedef StreamPlan<128, 1, 8, 1, 2, 4, 4> Whole1;    // (dense_item_192)
    typedef StreamPlan<128, 2, 4, 2, 1, 4, 4> Half;
    typedef StreamPlan<128, 1, 4, 2, 1, 4, 4> Quarter;
    static constexpr int LDS = Whole::LDS;
};
template <> struct DensePlan<64> {
    typedef StreamPlan<64, 4, 4, 1, 2, 4, 4> Whole;
    typedef StreamPlan<64, 4, 2, 2, 1, 4, 4> Half;
    typedef StreamPlan<64, 2, 2, 2, 1, 4, 4> Quarter;
    static constexpr int LDS = Whole::LDS;
};

// One wavefront's part of an item whose first query is q00: the queries from q0 on, stored up to `end`; `stage` bytes into the
// LDS its output goes through.
template <class P>
__device__ __forceinline__ void dense_wave(const AttnParams& p, char* lds, int pair, int q00, int q0, int end, int wave, int stage)
{
    typedef typename P::S S;
    constexpr int D = P::D;
    const int lane = threadIdx.x & 63;
    const int smp = p.H.of(pair), head = pair - smp * p.H.d;
    const int kv_len = valid_tokens(p, smp);
    const Rows Q = rows_of(p.q, p.in, smp, head, p.n0), K = rows_of(p.k, p.in, smp, head, p.n0);
    const Rows V = rows_of(p.v, p.in, smp, head, p.n0), O = rows_of(p.o, p.out, smp, head, p.n0);
    char* out_stage = lds + stage;
    StreamRegs<S, D> x;
    if (q00 >= kv_len) {                          // padding rows only: zero
        if (wave % P::WK != 0) return;
#pragma unroll
        for (int q = 0; q < S::NQ; ++q) x.ls[q][0] = 0.f;
        stream_output_rows<S, D>(x, O, q0, 0, end, lane, out_stage);
        return;
    }
    AllKeys<P> keys;
    const int last = ((kv_len + 31) / 32 + P::WK - 1) / P::WK - 1;
    stream_attend<P>(x, lds, Q, K, V, q0, kv_len, p.c, last, keys, wave, lane);
    __syncthreads();                              // every wavefront has read its last tile
    if constexpr (P::WK > 1) stream_merge_rows<P>(x, lds, O, q0, kv_len, end, wave, lane);
    else stream_output_rows<S, D>(x, O, q0, kv_len, end, lane, out_stage);
}
// A (sample, head)'s `tile` queries number item % nq, from `ahead` on.
template <class P>
__device__ __forceinline__ void dense_item(const AttnParams& p, char* lds, int item, int tile, int ahead)
{
    const int pair = p.nq.of(item), q00 = (item - pair * p.nq.d) * tile + ahead;
    if (q00 >= p.N) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    dense_wave<P>(p, lds, pair, q00, q00 + wave / P::WK * 16 * P::NQ, p.N, wave, wave * (16 * P::NQ * (P::D * 2 + 16)));
}

// 192 queries: the wavefronts of a SIMD take 32 and 16 (of 32 and 32, or none, a SIMD with two wavefronts would take as long
// as for 256); the same barriers and copies in both halves of the workgroup.
constexpr int DENSE_192 = 192;
template <class P, class P1>
__device__ __forceinline__ void dense_item_192(const AttnParams& p, char* lds, int pair, int q00, int end)
{
    static_assert(P::NW == 8 && P1::NW == 8 && P::NQ == 2 && P1::NQ == 1 && P::WK == 1 && P1::WK == 1, "");
    static_assert(P::UNROLL == P1::UNROLL && P::LC == P1::LC && P::LDS == P1::LDS, "the same barriers and copies");
    constexpr int ROW = P::D * 2 + 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave < 4) dense_wave<P>(p, lds, pair, q00, q00 + 32 * wave, end, wave, 32 * wave * ROW);
    else dense_wave<P1>(p, lds, pair, q00, q00 + 64 + 16 * wave, end, wave, (64 + 16 * wave) * ROW);
}

// Piece i of the pieces of 192 queries that items `first` .. `last` - 1 make, a (sample, head) at a time; without one, their number.
struct Piece192 {
    int bh, q0, end;                              // end: of the items' queries in this (sample, head)
    int n;
};
constexpr __host__ __device__ Piece192 piece_192(int i, int first, int last, int nq, int N)
{
    int n = 0;
    while (first < last) {
        const int at = first % nq, run = nq - at < last - first ? nq - at : last - first;
        const int q0 = at * DENSE_QT, end = (at + run) * DENSE_QT < N ? (at + run) * DENSE_QT : N;
        const int pieces = (end - q0 + DENSE_192 - 1) / DENSE_192;
        if (i < n + pieces) return {first / nq, q0 + (i - n) * DENSE_192, end, 0};
        n += pieces;
        first += run;
    }
    return {-1, 0, 0, n};
}

// The run of `chunk` items whose place `at` the workgroup's XCD works on.  Query tiles of the same (sample, head) share K and V
// in an XCD's L2, so runs are contiguous; the dispatcher deals consecutive workgroup ids out to the 8 XCDs in turn.  Samples of
// different length (turn > 0): the runs of one sample are those of neighbouring XCDs, so with every (sample, head)'s worth of
// places an XCD goes `turn` runs on, into another sample.  Which items are cut follows from their numbers as ever: how a query is
// computed does not hang on whether lengths were given.  us, turn = 0 / as it is, prompts of 1/B, 2/B, .. of the text tokens,
// H = 24: D = 64, B = 2, 1024 + 333 tokens 28.4 / 28.5, 2048 + 333 71.6 / 70.7; B = 8, 1024 + 333 91.2 / 83.9; B = 7, 512 + 500 49.0 /
// 45.5; D = 128, B = 2, 1024 + 512 57.3 / 54.4; B = 8, 512 + 512 86.8 / 75.2; B = 4, 4096 + 512 764 / 752; pairs that the XCDs do not
// divide: H = 7, B = 5, D = 64, 2048 + 500 55.0 / 52.9; B = 3, D = 128, 8192 + 512 588.9 / 589.2.
__device__ __forceinline__ int dense_run(const AttnParams& p, int at) { return (int)((blockIdx.x + (unsigned)(p.turn * p.nq.of(at))) % XCDS); }

// 256 queries of one (sample, head) per workgroup; the items of an XCD that do not fill its CUs evenly are
// cut into `cut` = 2 or 4 workgroups each, or into pieces of 192 queries (p.whole of an XCD's items stay whole).
template <int D>
__global__ __launch_bounds__(DensePlan<D>::Whole::NW * 64, 2) void attn_dense_stream_kernel(const AttnParams p)
{
    typedef DensePlan<D> DP;
    __shared__ __attribute__((aligned(1024))) char lds[DP::LDS];
    const int i = blockIdx.x / XCDS;
    if (i < p.whole) {
        const int item = dense_run(p, i) * p.chunk + i;
        if (item < p.items) dense_item<typename DP::Whole>(p, lds, item, DENSE_QT, 0);
        return;
    }
    if constexpr (D == 128) {
        if (p.cut == 3) {
            const int first = dense_run(p, p.whole) * p.chunk;
            const int last = first + p.chunk < p.items ? first + p.chunk : p.items;
            const Piece192 a = piece_192(i - p.whole, first + p.whole, last, p.nq.d, p.N);
            const int bh = __builtin_amdgcn_readfirstlane(a.bh), q0 = __builtin_amdgcn_readfirstlane(a.q0), end = __builtin_amdgcn_readfirstlane(a.end);
            if (bh >= 0) dense_item_192<typename DP::Whole, typename DP::Whole1>(p, lds, bh, q0, end);
            return;
        }
    }
    const int at = p.whole + (p.cut == 2 ? (i - p.whole) / 2 : (i - p.whole) / 4);
    const int item = dense_run(p, at) * p.chunk + at;
    if (item >= p.items) return;
    if (p.cut == 2) dense_item<typename DP::Half>(p, lds, item, DENSE_QT, (i - p.whole) % 2 * (DENSE_QT / 2));
    else dense_item<typename DP::Quarter>(p, lds, item, DENSE_QT, (i - p.whole) % 4 * (DENSE_QT / 4));
}

// Small problems: 32 queries per workgroup of 2 x 2 wavefronts.
template <int D>
__global__ __launch_bounds__(256, (D == 64 ? 4 : 2)) void attn_dense_pp_kernel(const AttnParams p)
{
    typedef StreamPlan<D, 1, 2, 2, 1, 2, 3> P;
    __shared__ __attribute__((aligned(1024))) char lds[P::LDS];
    const int at = blockIdx.x / XCDS, item = dense_run(p, at) * p.chunk + at;
    if (item < p.items) dense_item<P>(p, lds, item, P::QT, 0);
}

// ---------------------------------------------------------------------------
// Sparse path, 64-token mask tiles: one workgroup per (b, h, query-block) walks the kept list on the stream, a
// block per tile, the 64 keys of a block split between two groups of wavefronts that are merged at the end.
// Four wavefronts of 32 queries: 80 KB of stages at D = 128, two workgroups per CU and two wavefronts per SIMD; 40 KB at
// D = 64, three per CU (a wavefront of 64 queries there needs six registers more than there are).  One group of
// wavefronts per item instead would halve the rate of an item, and a row that keeps everything (the text rows) would be
// longer than its CU's share.  Copies are a whole step ahead and no more: stages for longer leads (4 of K and V) leave
// one workgroup per CU at D = 128 (1.2 to 1.7 times the time) and two at D = 64 (1.05 to 1.2 times); all copies at the
// head of the half step in which they are spread out: 1 to 1.5 % slower.
// us, B = 1, H = 24, no text rows, densities 0.1 / 0.3 / 1, two wavefront groups on alternating phases of 32x32x16 MFMAs behind two
// planner launches before and now: D = 128, N = 384 16.3 16.5 18.6 -> 7.5 9.2 11.4; 2816 56 90 221 -> 33 51 122; 8960 261 579
// 1727 -> 156 328 952; D = 64, N = 2816 27 43 106 -> 20 29 71.
// ---------------------------------------------------------------------------
template <int D> struct Sparse64Plan { typedef StreamPlan<128, 2, 2, 2, 1, 2, 3, 4, 4> P; };
template <> struct Sparse64Plan<64> { typedef StreamPlan<64, 2, 2, 2, 1, 2, 3, 4, 4> P; };

template <int D>
__global__ __launch_bounds__(Sparse64Plan<D>::P::NW * 64, (D == 64 ? 3 : 2)) void attn_sparse_pp_kernel(const AttnParams p)
{
    typedef typename Sparse64Plan<D>::P P;
    typedef typename P::S S;
    static_assert(P::QT == 64, "one item = 64 queries");
    __shared__ __attribute__((aligned(1024))) char lds[P::LDS];

    const auto work = sparse_work<64, 2>(p, lds + (P::NSK + P::NSV - 1) * P::TILE);    // (the last stage to be filled)
    const int item = work.rec.item;
    if (item < 0 || work.rec.nblk <= 0) leave_plan<64, 2>(p, work);
    if (item < 0) return;
    const int bh = p.nq.of(item);
    const int qi = item - bh * p.nq.d;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int smp = p.H.of(bh), head = bh - smp * p.H.d;
    const int kv_len = valid_tokens(p, smp);
    const Rows Q = rows_of(p.q, p.in, smp, head, p.n0), K = rows_of(p.k, p.in, smp, head, p.n0);
    const Rows V = rows_of(p.v, p.in, smp, head, p.n0), O = rows_of(p.o, p.out, smp, head, p.n0);
    const int q0 = qi * 64 + wave / P::WK * 16 * P::NQ;
    char* out_stage = lds + wave * (16 * P::NQ * (D * 2 + 16));
    const int n = work.rec.nblk;

    StreamRegs<S, D> x;
    if (n <= 0 || qi * 64 >= kv_len) {            // nothing kept, or padding rows only: the rows are zero
        if (n > 0) leave_plan<64, 2>(p, work);
        if (wave % P::WK != 0) return;
#pragma unroll
        for (int q = 0; q < P::NQ; ++q) x.ls[q][0] = 0.f;
        stream_output_rows<S, D>(x, O, q0, 0, p.N, lane, out_stage);
        return;
    }
    KeptTiles<P> keys(work.kept);
    stream_attend<P>(x, lds, Q, K, V, q0, kv_len, p.c, n - 1, keys, wave, lane);
    leave_plan<64, 2>(p, work);
    __syncthreads();                              // every wavefront has read its last tile
    stream_merge_rows<P>(x, lds, O, q0, kv_len, p.N, wave, lane);
}

// Partial result of one piece of a split item: the fp32 accumulators in register order
// ([wavefront][register pair][lane], 8 bytes each), then (m, l) per lane.
template <int D>
struct PartialSlot {
    static constexpr size_t ML_OFF = (size_t)4 * (D / 32) * 4 * 64 * 16;      // 64 KB | 32 KB
    static constexpr size_t BYTES = ML_OFF + 4 * 64 * 2 * 4;                  // + 2 KB
};

// ---------------------------------------------------------------------------
// Sparse path, 128-token mask tiles: one workgroup per plan record walks the kept-block list of its
// piece on the 16x16x32 stream, 128 queries in four wavefronts of 32 (D = 128, 64 KB of LDS, two workgroups
// per CU) or two of 64 (D = 64, 32 KB, four per CU): two wavefronts per SIMD, of different items, so the
// fixed cost of an item (list lookup, first copies, Q load, output) hides behind the neighbour's loop.
// us, B = 1, H = 24, D = 128 at densities 0.15 / 0.3 / 0.6, against 32x32x16 MFMAs alternating with softmax phases:
// N = 4480 70.6 -> 66.8, 97.9 -> 90.9, 157 -> 145; N = 8960 194 -> 180, 321 -> 285, 590 -> 521; N = 384 17.7 -> 16.3.
// ---------------------------------------------------------------------------
template <int D> struct SparsePlan { typedef StreamPlan<128, 2, 4, 1, 1, 4, 4> P; };
template <> struct SparsePlan<64> { typedef StreamPlan<64, 4, 2, 1, 1, 4, 4> P; };

template <int D>
__device__ __forceinline__ void sparse_stream_record(const AttnParams& p)
{
    typedef typename SparsePlan<D>::P P;
    typedef typename P::S S;
    static_assert(P::QT == 128, "one record = 128 queries");
    __shared__ __attribute__((aligned(1024))) char lds[P::LDS];

    constexpr int ROUNDS = D == 64 ? 0 : 2;       // (more than 2048 rows: run_sparse)
    const auto work = sparse_work<128, ROUNDS>(p, lds + (P::NSK + P::NSV - 1) * P::TILE);    // (the last stage to be filled)
    const PlanRec rec = work.rec;
    const int item = rec.item;
    if (rec.nblk <= 0) leave_plan<128, ROUNDS>(p, work);
    if (item < 0) return;
    const int bh = p.nq.of(item);
    const int qi = item - bh * p.nq.d;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int smp = p.H.of(bh), head = bh - smp * p.H.d;
    const int kv_len = valid_tokens(p, smp);
    const Rows Q = rows_of(p.q, p.in, smp, head, p.n0), K = rows_of(p.k, p.in, smp, head, p.n0);
    const Rows V = rows_of(p.v, p.in, smp, head, p.n0), O = rows_of(p.o, p.out, smp, head, p.n0);
    const int q0 = qi * 128 + wave * 16 * P::NQ;
    char* out_stage = lds + wave * (16 * P::NQ * (D * 2 + 16));

    StreamRegs<S, D> x;
    if (rec.nblk <= 0) {                          // nothing kept: the rows are zero
#pragma unroll
        for (int q = 0; q < P::NQ; ++q) x.ls[q][0] = 0.f;
        stream_output_rows<S, D>(x, O, q0, 0, p.N, lane, out_stage);
        return;
    }
    // Whole blocks: what lies at or beyond kv_len in a row's last block is masked, at most three steps.
    KeptKeys<P> keys(work.kept);
    stream_attend<P>(x, lds, Q, K, V, q0, kv_len, p.c, rec.nblk * 4 - 1, keys, wave, lane);
    leave_plan<128, ROUNDS>(p, work);
    __syncthreads();                              // every wavefront has read its last tile
    if (rec.w < 0) {                              // the whole item
        stream_output_rows<S, D>(x, O, q0, kv_len, p.N, lane, out_stage);
        return;
    }

    // ---- a piece of a split item: leave (acc, m, l) in this piece's slot; the piece that
    // finishes last adds all of them up, in piece order (so the sum does not depend on which
    // one that is).  A piece has at least one valid key per query, so every m is finite.
    // The slots are written and read with device-scope relaxed atomic accesses, each of which
    // is coherent across the chip by itself, instead of plain accesses between device-scope
    // fences: a release fence would write back every dirty line of the XCD's L2.  Order: a
    // wavefront's stores are acknowledged (vmcnt 0) before the barrier after which one thread
    // counts the piece in; the last piece reads only after it has seen the full count.
    typedef unsigned long long u64;
    constexpr size_t SLOT_BYTES = PartialSlot<D>::BYTES;
    constexpr int PAIRS = S::DT * S::NQ * 2;      // 64-bit words of accumulators per lane
    static_assert((size_t)P::NW * PAIRS * 64 * 8 == PartialSlot<D>::ML_OFF, "the slot holds the accumulators");
    const int pieces = (rec.w & 15) + 1;
    const int piece = (rec.w >> 4) & 15;
    const int slot0 = rec.w >> 8;
    auto slot_acc = [&](int k) -> u64* { return (u64*)(p.partial + (size_t)(slot0 + k) * SLOT_BYTES) + (size_t)wave * PAIRS * 64 + lane; };
    // (m, l) of query 16 q + n, held by the four lanes n, n + 16, ..: once per query
    auto slot_ml = [&](int k, int q) -> u64* {
        return (u64*)(p.partial + (size_t)(slot0 + k) * SLOT_BYTES + PartialSlot<D>::ML_OFF) + (wave * P::NQ + q) * 16 + (lane & 15);
    };
    {
        u64* pacc = slot_acc(piece);
#pragma unroll
        for (int i = 0; i < PAIRS; ++i) {
            const u64 v = (u64)__float_as_uint(x.acc[i / 8][i % 8 * 2]) | ((u64)__float_as_uint(x.acc[i / 8][i % 8 * 2 + 1]) << 32);
            __hip_atomic_store(pacc + i * 64, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (lane < 16) {
#pragma unroll
            for (int q = 0; q < P::NQ; ++q) {
                const u64 ml = (u64)__float_as_uint(x.m[q]) | ((u64)__float_as_uint(x.ls[q][0]) << 32);
                __hip_atomic_store(slot_ml(piece, q), ml, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    __shared__ int arrived_before;
    wait_vmcnt<0>();
    __syncthreads();
    if (tid == 0) arrived_before = __hip_atomic_fetch_add(&p.arrived[slot0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (arrived_before != pieces - 1) return;

#pragma unroll
    for (int q = 0; q < P::NQ; ++q) { x.m[q] = -INFINITY; x.ls[q][0] = 0.f; }
    for (int k = 0; k < pieces; ++k) {
#pragma unroll
        for (int q = 0; q < P::NQ; ++q) {
            const u64 ml = __hip_atomic_load(slot_ml(k, q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            x.m[q] = fmaxf(x.m[q], __uint_as_float((unsigned)ml));
        }
    }
#pragma unroll
    for (int b = 0; b < S::DT * S::NQ / 4; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) x.acc[b][r] = 0.f;
    for (int k = 0; k < pieces; ++k) {
        float a[P::NQ];
#pragma unroll
        for (int q = 0; q < P::NQ; ++q) {
            const u64 ml = __hip_atomic_load(slot_ml(k, q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            a[q] = __builtin_amdgcn_exp2f(__uint_as_float((unsigned)ml) - x.m[q]);
            x.ls[q][0] += __uint_as_float((unsigned)(ml >> 32)) * a[q];
        }
        const u64* pacc = slot_acc(k);
#pragma unroll
        for (int i = 0; i < PAIRS; ++i) {
            const u64 v = __hip_atomic_load(pacc + i * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            x.acc[i / 8][i % 8 * 2] += __uint_as_float((unsigned)v) * a[i / 2 % P::NQ];
            x.acc[i / 8][i % 8 * 2 + 1] += __uint_as_float((unsigned)(v >> 32)) * a[i / 2 % P::NQ];
        }
    }
    stream_output_rows<S, D>(x, O, q0, kv_len, p.N, lane, out_stage);
}

// ---------------------------------------------------------------------------
// Sparse path, 128-token mask tiles, D = 64, short calls: FOUR wavefronts of 32 queries per record, 32 KB of
// LDS, four workgroups per CU.  A step of its loop takes half as long as one of 64 queries per wavefront, which
// counts when every record is resident at once and the longest chain is the time.
//
// Per tile j two slots separated by workgroup barriers:
//   B(j)  softmax of S_j; copies of V_{j+1} and K_{j+2} issued; first V_j^T fragments requested
//   A(j)  O^T += V_j^T P_j^T ; S_{j+1} = K_{j+1} Q^T
// LDS: K stages 0,1 and V stages 2,3; tile t in stage t % 2.  When B(j) starts every
// wavefront has finished A(j-1), the last reader of V_{j-1} and K_j, whose stages take
// V_{j+1} and K_{j+2}.  Copies complete in issue order, so "all but the newest n" is a wait
// for everything older: K_{j+1} (issued in B(j-1)) is awaited at the end of B(j) with this
// slot's copies still in flight, V_{j+1} at the end of A(j) with K_{j+2} still in flight.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void sparse_short_record(const AttnParams& p)
{
    constexpr int D = 64;
    typedef Geo<D> G;
    constexpr int PD = 3;                         // (more does not fit 128 registers)
    typedef TileItems<D, PD> TI;
    constexpr int NW = 4, QT = 128, KS = D / 16, DB = D / 32;
    constexpr int LPT = G::LOADS / NW;            // copy instructions per wavefront per tile (K or V)

    __shared__ __attribute__((aligned(1024))) char lds[4 * G::TILE_BYTES];
    auto k_stage = [&](int t) -> char* { return lds + (t & 1) * G::TILE_BYTES; };
    auto v_stage = [&](int t) -> char* { return lds + (2 + (t & 1)) * G::TILE_BYTES; };

    auto work = sparse_work<128, 4>(p, v_stage(1));    // (the last stage to be filled)
    const PlanRec rec = work.rec;
    const int item = rec.item;
    if (rec.nblk <= 0) leave_plan<128, 4>(p, work);
    if (item < 0) return;
    const int bh = p.nq.of(item);
    const int qi = item - bh * p.nq.d;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31;
    const int h = lane >> 5;

    const int smp = p.H.of(bh), head = bh - smp * p.H.d;
    const int kv_len = valid_tokens(p, smp);
    const Rows Q = rows_of(p.q, p.in, smp, head, p.n0), K = rows_of(p.k, p.in, smp, head, p.n0);
    const Rows V = rows_of(p.v, p.in, smp, head, p.n0), O = rows_of(p.o, p.out, smp, head, p.n0);

    const int qrow = qi * QT + wave * 32 + n;
    const bool qvalid = qrow < kv_len;

    // 64-key tiles of this piece (two per kept 128-key block; the item's last block may have one)
    int T = rec.nblk * 2;
    if (rec.nblk > 0) {
        typedef const __attribute__((address_space(4))) int32_t* cptr_t;
        const int end = work.kept.list != nullptr ? ((cptr_t)work.kept.list)[rec.nblk - 1] : 63 - __builtin_clzll(work.kept.bits);
        if ((end * 2 + 1) * KT >= kv_len) T -= 1;
    }
    f32x16 acc[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    if (T <= 0) {                                 // nothing kept: the rows are zero
        write_output<D>(O, acc, 0.f, qrow, false, p.N, h);
        return;
    }
    // first keys of tiles j+1, j+2, j+3 (not used from tile T on)
    const int key0 = work.kept.next<false>() * 128;
    int kn1 = key0 + KT;
    int kn2 = work.kept.next<false>() * 128;
    int kn3 = kn2 + KT;

    // Q and K_0 first: S_0 needs only these; V_0 and K_1 land while it is computed.
    u32x4 qraw[KS];
    load_q_async<D>(Q, qrow, qvalid, h, qraw);
    issue_tile<D, NW, false>(K, key0, kv_len, k_stage(0), wave, lane);
    issue_tile<D, NW, true>(V, key0, kv_len, v_stage(0), wave, lane);
    if (1 < T) issue_tile<D, NW, false>(K, kn1, kv_len, k_stage(1), wave, lane);

    SoftmaxState sm;
    sm.m = -INFINITY;
    sm.l = 0.f;
    const int tr_row = (lane & 15) >> 2;
    const int tr_col = ((lane & 3) << 2) + (((lane >> 4) & 1) << 4);
    if (1 < T) wait_vmcnt<2 * LPT>();
    else wait_vmcnt<LPT>();
    bf16x8 qf[KS];
    q_arrived<D>(qraw, qvalid, qf);
    __syncthreads();

    TileCtx<D, PD> ctx;
    bf16x8 pb[4];
    f32x16 st[2];
    k_addresses<D>(k_stage(0), n, h, ctx);
    items_prefetch<D, PD, TI::NPV, TI::NI>(ctx);
    items_run<D, PD, TI::NPV, TI::NI>(ctx, pb, qf, acc, st);   // S_0
    mask_tail(st, key0, kv_len, h);
    if (1 < T) wait_vmcnt<LPT>();                 // V_0 landed (K_1 may still be on its way)
    else wait_vmcnt<0>();

    for (int j = 0; j < T; ++j) {
        phase_barrier();                          // A(j-1) (or S_0) finished by every wavefront; V_j landed

        // ---- B(j)
        if (j + 1 < T) issue_tile<D, NW, true>(V, kn1, kv_len, v_stage(j + 1), wave, lane);
        if (j + 2 < T) issue_tile<D, NW, false>(K, kn2, kv_len, k_stage(j), wave, lane);
        v_addresses<D>(v_stage(j), h, tr_row, tr_col, ctx.vaddr);
        softmax_tile<D>(st, acc, sm, p.c, j == 0, pb);
        pin_in_phase(pb, sm.l);
        items_prefetch<D, PD, 0, TI::NI>(ctx);        // first V_j^T fragments of A(j)
        if (j + 2 < T) wait_vmcnt<2 * LPT>();     // K_{j+1} landed
        else if (j + 1 < T) wait_vmcnt<LPT>();
        else wait_vmcnt<0>();
        phase_barrier();

        // ---- A(j): PV(j) then QK(j+1) as one stream (without a tile j+1 the QK half re-reads
        // K_j, which is still in its stage, and its result is never used)
        __builtin_amdgcn_s_setprio(3);
        k_addresses<D>(k_stage((j + 1 < T) ? j + 1 : j), n, h, ctx);
        items_run<D, PD, 0, TI::NI>(ctx, pb, qf, acc, st);
        mask_tail(st, kn1, kv_len, h);
        __builtin_amdgcn_s_setprio(0);
        if (j + 2 < T) wait_vmcnt<LPT>();         // V_{j+1} landed
        else wait_vmcnt<0>();
        kn1 = kn2; kn2 = kn3;
        kn3 = (j & 1) == 0 ? work.kept.next<false>() * 128 : kn3 + KT;
    }

    leave_plan<128, 4>(p, work);
    // Output straight from registers: with four workgroups on the CU, row-wise through LDS was 2-3 % slower.
    if (rec.w < 0) {                              // the whole item
        write_output<D>(O, acc, sm.l, qrow, qvalid, p.N, h);
        return;
    }

    // ---- a piece of a split item: leave (acc, m, l) in this piece's slot; the piece that
    // finishes last adds all of them up, in piece order (so the sum does not depend on which
    // one that is).  A piece has at least one valid key per query, so every m is finite.
    // The slots are written and read with device-scope relaxed atomic accesses, each of which
    // is coherent across the chip by itself, instead of plain accesses between device-scope
    // fences: a release fence would write back every dirty line of the XCD's L2.  Order: a
    // wavefront's stores are acknowledged (vmcnt 0) before the barrier after which one thread
    // counts the piece in; the last piece reads only after it has seen the full count.
    typedef unsigned long long u64;
    constexpr size_t SLOT_BYTES = PartialSlot<D>::BYTES;
    constexpr int PAIRS = DB * 8;                 // 64-bit words of accumulators per lane
    const int P = (rec.w & 15) + 1;
    const int piece = (rec.w >> 4) & 15;
    const int slot0 = rec.w >> 8;
    auto slot_acc = [&](int k) -> u64* { return (u64*)(p.partial + (size_t)(slot0 + k) * SLOT_BYTES) + (size_t)wave * PAIRS * 64 + lane; };
    auto slot_ml = [&](int k) -> u64* { return (u64*)(p.partial + (size_t)(slot0 + k) * SLOT_BYTES + PartialSlot<D>::ML_OFF) + wave * 64 + lane; };
    {
        u64* pacc = slot_acc(piece);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const u64 v = (u64)__float_as_uint(acc[db][2 * j]) | ((u64)__float_as_uint(acc[db][2 * j + 1]) << 32);
                __hip_atomic_store(pacc + (db * 8 + j) * 64, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        const u64 ml = (u64)__float_as_uint(sm.m) | ((u64)__float_as_uint(sm.l) << 32);
        __hip_atomic_store(slot_ml(piece), ml, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __shared__ int arrived_before;
    wait_vmcnt<0>();
    __syncthreads();
    if (tid == 0) arrived_before = __hip_atomic_fetch_add(&p.arrived[slot0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (arrived_before != P - 1) return;

    float m = -INFINITY;
    for (int k = 0; k < P; ++k) {
        const u64 ml = __hip_atomic_load(slot_ml(k), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        m = fmaxf(m, __uint_as_float((unsigned)ml));
    }
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    float l = 0.f;
    for (int k = 0; k < P; ++k) {
        const u64 ml = __hip_atomic_load(slot_ml(k), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float a = __builtin_amdgcn_exp2f(__uint_as_float((unsigned)ml) - m);
        l += __uint_as_float((unsigned)(ml >> 32)) * a;
        const u64* pacc = slot_acc(k);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const u64 v = __hip_atomic_load(pacc + (db * 8 + j) * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                acc[db][2 * j] += __uint_as_float((unsigned)v) * a;
                acc[db][2 * j + 1] += __uint_as_float((unsigned)(v >> 32)) * a;
            }
    }
    write_output<D>(O, acc, l, qrow, qvalid, p.N, h);
}

// The record of a workgroup on the kernel of its head size and length.
template <int D>
__global__ __launch_bounds__(256, (D == 64 ? 4 : 2)) void attn_sparse_sg_kernel(const AttnParams p)
{
    if constexpr (D == 64) sparse_short_record(p);
    else sparse_stream_record<D>(p);
}
__global__ __launch_bounds__(SparsePlan<64>::P::NW * 64, 2) void attn_sparse_wide_kernel(const AttnParams p)
{
    sparse_stream_record<64>(p);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct WorkspaceLayout {
    size_t counts_off, order_off, index_off, arrived_off, partial_off, total;
    int chunk;    // plan entries per XCD
    int pmax;     // partial-result slots per segment (128-token tiles)
};

// items of one XCD: (b,h) pairs are dealt round-robin over the XCDs
inline int plan_items(int B, int H, int nb) { return ((B * H + XCDS - 1) / XCDS) * nb; }

// 64-token tiles:  counts | order int32[8*chunk]   | index
// 128-token tiles: counts | records PlanRec[8*chunk] | index | arrived int32[8*pmax] | partial slots [8*pmax]
// `slots` < 0: min(256, items) partial-result slots per segment; otherwise that many at most.  The split rule may ask for
// more (an item that gets none stays whole): of rows by length it cuts a few, of rows all alike up to every one.
inline WorkspaceLayout workspace_layout(int B, int H, int nb, int D, int block, int slots = -1)
{
    const size_t rows = (size_t)B * H * nb;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    WorkspaceLayout w;
    const int items = plan_items(B, H, nb);
    w.counts_off = 0;
    w.order_off = up(rows * 4);
    if (block == 128) {
        w.pmax = SPLIT_SLOTS < items ? SPLIT_SLOTS : items;
        if (slots >= 0 && slots < w.pmax) w.pmax = slots;
        w.chunk = items + w.pmax;
        w.index_off = w.order_off + up((size_t)XCDS * w.chunk * sizeof(PlanRec));
        w.arrived_off = w.index_off + up(rows * (size_t)nb * 4);
        w.partial_off = w.arrived_off + up((size_t)XCDS * w.pmax * 4);
        const size_t slot = D == 64 ? PartialSlot<64>::BYTES : PartialSlot<128>::BYTES;
        w.total = w.partial_off + up((size_t)XCDS * w.pmax * slot);
    } else {
        w.pmax = 0;
        w.chunk = items;
        w.index_off = w.order_off + up((size_t)XCDS * w.chunk * 4);
        w.arrived_off = w.partial_off = w.total = w.index_off + up(rows * (size_t)nb * 4);
    }
    return w;
}

int check_common(const void* q, const void* k, const void* v, const void* o,
                 int B, int H, int N, int D, int kv_len)
{
    if (!q || !k || !v || !o) return RAPID_ERR_NULL;
    if (B <= 0 || H <= 0 || N <= 0) return RAPID_ERR_SHAPE;
    if (kv_len < 1 || kv_len > N) return RAPID_ERR_SHAPE;
    if ((long long)B * H > 0x7fffffffLL / 4096) return RAPID_ERR_SHAPE;
    if (N > (1 << 22)) return RAPID_ERR_SHAPE;
    if (D != 64 && D != 128) return RAPID_ERR_UNSUPPORTED;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return RAPID_ERR_ALIGN;
    // O is written while other workgroups still read Q, K and V: it must not share a byte with them
    const uintptr_t bytes = (uintptr_t)B * H * N * D * 2, ob = (uintptr_t)o;
    for (const void* in : {q, k, v}) {
        const uintptr_t ib = (uintptr_t)in;
        if (ob < ib + bytes && ib < ob + bytes) return RAPID_ERR_ALIAS;
    }
    return RAPID_OK;
}

// One validated call: tensors as segment views, sizes, lengths.
struct Problem {
    SegTensor q, k, v, o;
    SegStrides in, out;
    int n0;
    int B, H, N, D;
    int kv_len;
    const int32_t* kv_lens;
    float scale;
};

void fill_common(AttnParams& p, const Problem& pr)
{
    p.q = pr.q; p.k = pr.k; p.v = pr.v; p.o = pr.o;
    p.in = pr.in; p.out = pr.out;
    p.kv_lens = pr.kv_lens;
    p.n0 = pr.n0;
    p.H = divisor(pr.H, (long long)pr.B * pr.H);
    p.N = pr.N; p.kv_len = pr.kv_len;
    p.c = pr.scale * LOG2E;
}

int run_dense(const Problem& pr, void* stream)
{
    AttnParams p{};
    fill_common(p, pr);
    p.turn = pr.kv_lens == nullptr || pr.B == 1 ? 0 : pr.B < XCDS ? XCDS / pr.B : 1;
    hipStream_t s = (hipStream_t)stream;
    const long long pairs = (long long)pr.B * pr.H, small = pairs * ((pr.N + 31) / 32);
    const long long items = pairs * ((pr.N + DENSE_QT - 1) / DENSE_QT), chunk = (items + XCDS - 1) / XCDS;
    // of these, the ones with valid rows (padding costs next to nothing)
    const long long small_live = pairs * ((pr.kv_len + 31) / 32);
    const long long live = (pairs * ((pr.kv_len + DENSE_QT - 1) / DENSE_QT) + XCDS - 1) / XCDS;
    // 32 queries per workgroup: while they are resident at once the shortest chain of steps per wavefront wins, as long
    // as the other kernel has too few queries per workgroup to choose from.  us, this kernel / the other, H heads, B = 1:
    //   N <= 64: three quarters of 256 queries do not exist (B = 64, H = 38, N = 64: 20.0 / 31.6 at D = 64, 45 / 61 at 128)
    //   D = 64: N = 1024, H = 24 15.0 / 15.3; 2048, 12 23.5 / 23.6; past three quarters of the 1024 places the quarters of
    //     the other win: 1152, 24 19.4 / 16.1; 2048, 16 29.6 / 25.0; so they do over many keys: 16384, 1 110 / 108
    //   D = 64 again where the other has more than one place per quarter (over 16 items of an XCD): 320, 96 10.0 / 10.7;
    //     1024, 38 22.2 / 23.5; 1361, 24 27.1 / 27.9; but 384, 96 12.8 / 11.9; 512, 80 at 400 keys 13.8 / 12.6; 1792, 24
    //     36.8 / 34.5
    //   D = 128: N = 640, H = 24 13.3 / 15.6; its 16-query wavefronts read K and V from LDS twice as often per product and
    //     it loses on long sequences: 8192, 2 93 / 79
    const long long places = (pr.D == 64 ? 4 : 2) * XCDS * CUS_PER_XCD;
    const bool short_chain = pr.N <= 64 ||
        (pr.D == 128 ? small <= places && pr.N <= 1024
                     : (small_live <= places * 3 / 4 && small <= places && pr.kv_len <= 8192) ||
                       (chunk > CUS_PER_XCD / 2 && pr.kv_len <= 2048 && small <= (pr.N >= 640 ? places * 5 / 4 : places)));
    if (short_chain) {
        p.nq = divisor((pr.N + 31) / 32, small);
        p.items = (int)small;
        p.chunk = (p.items + XCDS - 1) / XCDS;
        const dim3 grid((unsigned)p.chunk * XCDS);
        if (pr.D == 64) hipLaunchKernelGGL((attn_dense_pp_kernel<64>), grid, dim3(256), 0, s, p);
        else hipLaunchKernelGGL((attn_dense_pp_kernel<128>), grid, dim3(256), 0, s, p);
        return hipGetLastError() == hipSuccess ? RAPID_OK : RAPID_ERR_DEVICE;
    }
    p.nq = divisor((pr.N + DENSE_QT - 1) / DENSE_QT, items);
    if (items > 0x7fffffffLL / 8) return RAPID_ERR_SHAPE;
    p.items = (int)items;
    p.chunk = (int)chunk;
    // What is left over after every CU of an XCD got the same number of items is cut so that it still makes
    // one workgroup per CU at most: a last round of an eighth of the CUs takes a quarter of the time.  us, items of an
    // XCD: 33 (H = 24, N = 2816) whole 136, in 2 116, in 4 105 at D = 128, 81 / 60 / 55 at D = 64; 198 (N = 16896)
    // 2875 / 2734 / 2703; 108 (B = 2, N = 4429, D = 64) 257 / 231 / 257.  More than half of a round is not cut in two: 54
    // items (N = 4608) 218 / 247 / 255.  At D = 128 up to three quarters of a round make pieces of 192 queries, still one per CU
    // at most (the rest of one (sample, head) after the other, so a few more than 4 for 3 items).  us, whole / 192: 18 items
    // (H = 24, N = 1536) 42.1 / 38.2; 20 (B = 4, H = 2, N = 5000) 98.1 / 91.8; 24 (N = 1800) 46.4 / 43.7; 54 (N = 4608) 212.9 /
    // 211.8; 84 (N = 7168) 473 / 466; 147 (N = 12544) 1399 / 1380: after full rounds the chip is warm and its clock gives
    // most of it back.
    // D = 64, no full round: two workgroups share a CU, so quarters fill it up to 16 items (with valid rows) and win up to
    // 24, halves up to 32, once the sequence is long enough to pay for more prologues.  us, whole / 2 / 4, H heads: N =
    // 1152, 24 (14 items) - / 18.3 / 16.1; 1792, 24 (21) 36.0 / 35.1 / 34.5; 2048, 24 40.2 / 38.9 / 38.9; 2304, 24 (27)
    // 44.4 / 43.1 / 49.5; 2560, 24 (30) 48.7 / 48.1 / 55.3; of shorter ones 1024, 64 (32) 23.4 / 24.1 / 27.7; 512, 96 (24)
    // 14.9 / 16.5 / 16.0; 256, 256 (32) 11.0 / 13.2 / 15.0; 858 keys of 2560, 24 (30, 12 of them with valid rows) 19.7 /
    // 15.8 / -; 250 of 320, 128 (32, 16) 10.4 / 12.7 / 12.8.
    const bool one_round = pr.D == 64 && p.chunk <= CUS_PER_XCD;
    const int rest = one_round ? p.chunk : p.chunk % CUS_PER_XCD;
    const bool fits = rest <= CUS_PER_XCD / 2 || (live <= CUS_PER_XCD / 2 && pr.kv_len >= 640);
    p.cut = one_round ? (fits ? 4 : pr.kv_len < 1280 ? 1 : live <= 24 ? 4 : 2) : rest * 4 <= CUS_PER_XCD ? 4 : rest * 2 <= CUS_PER_XCD ? 2 : 1;
    p.whole = p.cut == 1 ? p.chunk : p.chunk - rest;
    int groups = p.whole + (p.chunk - p.whole) * p.cut;
    if (pr.D == 128 && p.cut == 1 && rest > CUS_PER_XCD / 2 && rest <= CUS_PER_XCD * 3 / 4) {
        int pieces = 0;
        for (int x = 0; x < XCDS; ++x) {
            const int first = x * p.chunk, last = first + p.chunk < p.items ? first + p.chunk : p.items;
            const int n = piece_192(0x7fffffff, first + p.chunk - rest, last, p.nq.d, p.N).n;
            pieces = n > pieces ? n : pieces;
        }
        if (pieces <= CUS_PER_XCD) { p.cut = 3; p.whole = p.chunk - rest; groups = p.whole + pieces; }
    }
    const dim3 grid((unsigned)groups * XCDS);
    if (pr.D == 64) hipLaunchKernelGGL((attn_dense_stream_kernel<64>), grid, dim3(DensePlan<64>::Whole::NW * 64), 0, s, p);
    else hipLaunchKernelGGL((attn_dense_stream_kernel<128>), grid, dim3(DensePlan<128>::Whole::NW * 64), 0, s, p);
    return hipGetLastError() == hipSuccess ? RAPID_OK : RAPID_ERR_DEVICE;
}

// nb = ceil(N / block): the last mask block may be ragged (it then ends at N)
// `mask` null: counts and lists are already in the workspace (written by the selection kernels)
int run_sparse(const Problem& pr, int block, const unsigned char* mask, void* workspace, size_t workspace_bytes,
               void* stream, int slots = -1)
{
    const int B = pr.B, H = pr.H, N = pr.N, D = pr.D;
    const int nb = (N + block - 1) / block;
    const long long rows = (long long)B * H * nb;
    if (rows > 0x7fffffffLL / 16) return RAPID_ERR_SHAPE;
    const WorkspaceLayout w = workspace_layout(B, H, nb, D, block, slots);
    if (!workspace || workspace_bytes < w.total) return RAPID_ERR_WORKSPACE;
    if (!aligned16(workspace)) return RAPID_ERR_ALIGN;

    char* ws = (char*)workspace;
    int32_t* counts = (int32_t*)(ws + w.counts_off);
    int32_t* order = (int32_t*)(ws + w.order_off);
    int32_t* index = (int32_t*)(ws + w.index_off);
    hipStream_t s = (hipStream_t)stream;

    const int xcd_items = plan_items(B, H, nb);
    int32_t* arrived = (int32_t*)(ws + w.arrived_off);
    // All rows on the chip at once and none that could be cut: no plan, every workgroup finds its row by itself.  us, plan
    // launches / without: H = 2, N = 256 16.5 / 10.5; D = 64, H = 4, N = 2048 under 64-token masks 15.4 / 10.2 (density 0.1),
    // 23.6 / 18.5 (all ones); B = 2, H = 24, N = 1024 under 64-token masks, D = 64, 768 rows 18.3 / 15 (0.3).
    // More rows than that, and long ones: the order of a plan is worth more than its launch, most of all where samples differ.  us,
    // without a plan / with, densities 0.15, 0.7 and by sample 1 0.5 0.3 0.15 in turn, rows of an XCD, blocks of a row:
    //   128-token masks, D = 64: 54 x 6 18.9 18.9 18.6 / 22.3 22.9 22.1, 126 x 6 31.5 35.2 35.1 / 34.3 39.2 36.8; 64 x 8 23.2 24.9
    //     23.0 / 26.4 27.7 26.4, 72 x 8 25.9 30.7 30.9 / 27.4 30.9 28.7, 104 x 8 34.2 39.9 40.4 / 31.7 40.3 36.0; 60 x 15 33.9 36.3
    //     34.5 / 37.2 40.0 37.7, 75 x 15 38.6 48.8 45.8 / 38.8 45.8 42.2, 120 x 15 48.2 65.6 58.3 / 44.2 64.0 56.2: a line at two
    //     rows per CU, and at 6 blocks
    //   64-token masks, D = 64: 96 x 16 17.3 20.4 21.0 / 18.4 22.6 21.1; 60 x 20 17.5 17.7 17.5 / 18.1 19.8 18.4, 80 x 20 19.8 22.5
    //     22.3 / 18.7 23.3 20.2; 64 x 32 21.7 23.8 24.7 / 22.9 24.5 27.9, 96 x 32 24.3 31.5 31.5 / 24.2 32.5 31.0; 80 x 40 27.5 35.6
    //     38.4 / 27.4 34.8 34.5: two rows per CU, and 16 blocks
    //   D = 128: 128-token masks 40 x 10 29.9 33.1 33.1 / 32.0 34.2 32.5, 60 x 15 42.1 51.8 49.5 / 44.3 52.4 47.8 (up to 15 blocks
    //     there is none to cut); 64-token masks 48 x 24 25.4 27.9 28.6 / 26.5 28.0 28.1, 40 x 40 33.3 37.5 (0.3 34.7) / 34.0 36.4
    //     (34.5): one row per CU, and 24 blocks
    // (Rows dealt out over several XCDs: not told apart.)
    const bool short_rows = D == 128 ? block == 128 || nb <= 24 : nb <= (block == 128 ? 6 : 16);
    const int places = segment_cus(B * H, nb, block) * (block == 64 ? (D == 128 ? 2 : 3) : (D == 128 ? 2 : 4));
    const bool planned = xcd_items > places || (block == 128 && nb >= 2 * SPLIT_MIN_BLOCKS) ||
                         (xcd_items > CUS_PER_XCD * (D == 128 ? 1 : 2) && !short_rows && segments(B * H, nb, block) == XCDS);
    const long long mask_pieces = nb <= SMALL_NB ? (long long)(xcd_items / nb) * (((nb * nb + 7) / 8 + 3) / 4 * 4) : 0;
    const bool small = nb <= SMALL_NB && xcd_items <= SMALL_ITEMS && mask_pieces <= SMALL_PIECES;
    // Every workgroup looks its row up by itself, while a place works through few of them and (128-token masks) no row is
    // long enough to be cut.  us, plan launch / looked up, 64-token masks, H = 24 unless said otherwise, rows of an XCD x blocks: D = 128 (64 places) 96 x 32 30.3 / 28.1; 132 x 44 62.4 / 61.9; 192 x 64
    // 92.0 / 93.2; B = 8, 240 x 10 42.0 / 42.6; D = 64 (96 places) 96 x 32 23.0 / 20.7; 132 x 44 38.9 / 36.9; 192 x 64 56.6 / 54.5; B = 4,
    // 192 x 16 25.9 / 24.3; B = 8, 240 x 10 23.0 / 21.5; with 2 or 3 pairs the same within 0.5 %.
    // 128-token masks, density 0.2: D = 128 96 x 8 27.4 / 24.4; 90 x 15 45.5 / 42.5; 144 x 12 51.5 / 49.9; 192 x 12 68.6 / 68.3; 216 x 9
    // 65.4 / 63.9 but 228 x 12 76.2 / 77.0; D = 64 96 x 8 19.2 / 15.1; 90 x 15 38.4 / 34.6; 192 x 12 40.7 / 39.2; 228 x 12 44.6 / 42.2.
    const bool found = planned && nb >= 8 && (block == 64 ? nb <= SMALL_NB : nb < 2 * SPLIT_MIN_BLOCKS) &&
                       xcd_items <= (D == 64 ? FOUND_ROWS : block == 64 ? 144 : 192) && (H == 1 || divisor(H, (long long)B * H).magic != 0u);
    const bool lists = mask != nullptr && (planned && !found ? !small : nb > SMALL_NB);      // compacted by a kernel of its own
    if (lists)
        hipLaunchKernelGGL(compact_mask_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s,
                           mask, (int)rows, nb, block, pr.kv_len, pr.kv_lens, H * nb, N, counts, index);
    if (lists && hipGetLastError() != hipSuccess) return RAPID_ERR_DEVICE;
    if (planned && small && !found) {
        // (the instructions of this kernel are fetched anew in every call: a third of the code, 6.3 -> 5.2 us at H = 24, N = 4608)
        const bool one = xcd_items <= 1024 && mask_pieces <= 4096;
        const auto kernel = block == 128 ? (one ? plan_small_kernel<true, 1, 4> : plan_small_kernel<true, SMALL_PER_THREAD, SMALL_PIECES / 1024>)
                                         : (one ? plan_small_kernel<false, 1, 4> : plan_small_kernel<false, SMALL_PER_THREAD, SMALL_PIECES / 1024>);
        hipLaunchKernelGGL(kernel, dim3(XCDS), dim3(1024), 0, s, mask, pr.kv_lens, pr.kv_len, N, block,
                           H, B * H, nb, w.chunk, w.pmax, D, counts, order, arrived);
    }
    else if (planned && !found && block == 128)
        hipLaunchKernelGGL(plan_split_kernel, dim3(XCDS), dim3(1024), 0, s, counts, B * H, nb, w.chunk,
                           w.pmax, D, (PlanRec*)order, arrived);
    else if (planned && !found)
        hipLaunchKernelGGL(plan_kernel, dim3(XCDS), dim3(1024), 0, s, counts, B * H, nb, w.chunk, order);
    if (hipGetLastError() != hipSuccess) return RAPID_ERR_DEVICE;

    AttnParams p{};
    fill_common(p, pr);
    p.mask = lists ? nullptr : mask;
    p.counts = counts; p.order = order; p.index = index;
    p.planned = found ? PLAN_FOUND : planned ? PLAN_READ : PLAN_NONE;
    p.pairs = B * H;
    p.segs = segments(B * H, nb, block);
    p.seg_magic = 0xffffffffu / (unsigned)p.segs + 1u;
    p.arrived = arrived;
    p.pmax = w.pmax;
    p.partial = ws + w.partial_off;
    // (dividends: items, and where every workgroup plans for itself its number in the segment, turned on: see sparse_work)
    p.nq = divisor(nb, rows + w.chunk + (long long)(w.chunk / CUS_PER_XCD + 1) * (3 * nb + 7));
    p.items = (int)rows;
    p.chunk = w.chunk;
    p.nb = nb;
    const dim3 grid((unsigned)w.chunk * XCDS);
    if (block == 128) {
        // D = 64: 64 queries per wavefront read LDS half as often, but a record takes longer; it wins where every place
        // of the chip (four per CU) gets at least two records.  us, 32 / 64 queries per wavefront, H = 24, densities 0.15 to 1:
        // 3072 rows (B = 8, N = 2048) 87 / 84 to 218 / 208; 6720 (B = 8, N = 4480) 267 / 267 to 973 / 939; 1536 rows
        // (B = 8, N = 1024) 41 / 42 to 67 / 74; 840 rows of N = 896 26.4 / 29.7.  Rows of one or two kept blocks are all
        // fixed cost, of which two wavefronts hide less than four: density 0.1, B = 8, H = 38, N = 896 36.5 / 38.3, 1152
        // 46.8 / 47.2, 1408 55.4 / 56.2 (0.3: 80.7 / 79.4; 1.0: 184 / 171), so not at 8 blocks per side and fewer; a mask of
        // the diagonal alone, which the host cannot tell, is 7 % slower on it at any N (B = 4, H = 24, N = 4480 46.1 / 49.5).
        // Calls of 840 to 2048 rows of more than 8 blocks would be up to 8 % faster on it, at errors against 64 bits 0.1 to 0.9 % larger
        // (2.320 / 2.326e-3 at 24 x 35, density 0.25): not taken.
        // (that many rows of more than 8 blocks always have a plan)
        if (D == 64 && rows > 2 * 4 * XCDS * CUS_PER_XCD && nb > 8 && p.planned == PLAN_READ) hipLaunchKernelGGL(attn_sparse_wide_kernel, grid, dim3(SparsePlan<64>::P::NW * 64), 0, s, p);
        else if (D == 64) hipLaunchKernelGGL((attn_sparse_sg_kernel<64>), grid, dim3(256), 0, s, p);
        else hipLaunchKernelGGL((attn_sparse_sg_kernel<128>), grid, dim3(SparsePlan<128>::P::NW * 64), 0, s, p);
    } else {
        if (D == 64) hipLaunchKernelGGL((attn_sparse_pp_kernel<64>), grid, dim3(Sparse64Plan<64>::P::NW * 64), 0, s, p);
        else hipLaunchKernelGGL((attn_sparse_pp_kernel<128>), grid, dim3(Sparse64Plan<128>::P::NW * 64), 0, s, p);
    }
    return hipGetLastError() == hipSuccess ? RAPID_OK : RAPID_ERR_DEVICE;
}

Problem contiguous_problem(const void* q, const void* k, const void* v, void* o, int B, int H, int N, int D,
                           int kv_len, float scale)
{
    Problem pr;
    auto whole = [](const void* ptr) { return SegTensor{(const __bf16*)ptr, (const __bf16*)ptr}; };
    pr.q = whole(q); pr.k = whole(k); pr.v = whole(v); pr.o = whole(o);
    pr.in = pr.out = {(long long)H * N * D, 0, (long long)N * D, D};
    pr.n0 = N;
    pr.B = B; pr.H = H; pr.N = N; pr.D = D;
    pr.kv_len = kv_len; pr.kv_lens = nullptr;
    pr.scale = scale > 0.f ? scale : 1.0f / sqrtf((float)D);
    return pr;
}

// The segments of rapid_attn_joint as a validated Problem.
int joint_problem(const rapid_attn_segment* segments, int n_segments, int B, int H, int D, int block, bool sparse,
                  int kv_len, const int* kv_lens, float scale, Problem& pr)
{
    if (!segments) return RAPID_ERR_NULL;
    if (n_segments != 1 && n_segments != 2) return RAPID_ERR_SHAPE;
    if (B <= 0 || H <= 0) return RAPID_ERR_SHAPE;
    if (D != 64 && D != 128) return RAPID_ERR_UNSUPPORTED;
    if (sparse && block != 64 && block != 128) return RAPID_ERR_UNSUPPORTED;
    long long N = 0;
    rapid_attn_segment seg[2];                    // strides of size-1 dimensions are not looked at
    for (int i = 0; i < n_segments; ++i) seg[i] = rapid_internal::normalised_segment(segments[i], B, H, i == 1 ? &seg[0] : nullptr);
    segments = seg;
    for (int i = 0; i < n_segments; ++i) {
        const rapid_attn_segment& g = segments[i];
        if (!g.q || !g.k || !g.v || !g.o) return RAPID_ERR_NULL;
        if (g.n <= 0) return RAPID_ERR_SHAPE;
        if (!aligned16(g.q) || !aligned16(g.k) || !aligned16(g.v) || !aligned16(g.o)) return RAPID_ERR_ALIGN;
        const long long st[6] = {g.in_stride_b, g.in_stride_h, g.in_stride_n, g.out_stride_b, g.out_stride_h, g.out_stride_n};
        for (int j = 0; j < 6; ++j) {
            if (st[j] < 0 || st[j] > (1LL << 40)) return RAPID_ERR_SHAPE;
            if (st[j] % 8 != 0) return RAPID_ERR_ALIGN;            // every row starts on 16 bytes
        }
        // rows are D contiguous elements; the bytes of 128 rows, which one copy descriptor spans, come to 2^31 at most (32 bits, unsigned)
        if (g.in_stride_n < D || g.out_stride_n < D || g.in_stride_n > (1LL << 23) || g.out_stride_n > (1LL << 23)) return RAPID_ERR_SHAPE;
        N += g.n;
    }
    if (N > (1 << 22)) return RAPID_ERR_SHAPE;
    if ((long long)B * H > 0x7fffffffLL / 4096) return RAPID_ERR_SHAPE;
    if (n_segments == 2) {
        // tiles of 64 keys and mask blocks of 128 queries must not straddle the two tensors
        if (segments[0].n % 128 != 0) return RAPID_ERR_SHAPE;
        if (segments[0].in_stride_h != segments[1].in_stride_h || segments[0].in_stride_n != segments[1].in_stride_n ||
            segments[0].out_stride_h != segments[1].out_stride_h || segments[0].out_stride_n != segments[1].out_stride_n)
            return RAPID_ERR_SHAPE;
    }
    if (kv_len == 0) kv_len = (int)N;
    if (kv_len < 1 || kv_len > N) return RAPID_ERR_SHAPE;

    auto view = [&](int which) {
        SegTensor t;
        const rapid_attn_segment& a = segments[0];
        const rapid_attn_segment* b2 = n_segments == 2 ? &segments[1] : nullptr;
        const void* p0 = which == 0 ? a.q : which == 1 ? a.k : which == 2 ? a.v : (const void*)a.o;
        const void* p1 = !b2 ? p0 : which == 0 ? b2->q : which == 1 ? b2->k : which == 2 ? b2->v : (const void*)b2->o;
        t.seg0 = (const __bf16*)p0; t.seg1 = (const __bf16*)p1;
        return t;
    };
    pr.q = view(0); pr.k = view(1); pr.v = view(2); pr.o = view(3);
    const rapid_attn_segment& a = segments[0];
    const rapid_attn_segment& b = segments[n_segments - 1];
    pr.in = {a.in_stride_b, b.in_stride_b, a.in_stride_h, a.in_stride_n};
    pr.out = {a.out_stride_b, b.out_stride_b, a.out_stride_h, a.out_stride_n};
    pr.n0 = n_segments == 2 ? segments[0].n : (int)N;
    pr.B = B; pr.H = H; pr.N = (int)N; pr.D = D;
    pr.kv_len = kv_len; pr.kv_lens = kv_lens;
    pr.scale = scale > 0.f ? scale : 1.0f / sqrtf((float)D);
    return RAPID_OK;
}

// The scratch of rapid_attn_block_sparse_static: one array per GPU, part of the loaded code
// object, alive until the process ends.  In host code `scratch` is only a handle for
// hipGetSymbolAddress; the device address is looked up once per device, with that device
// current, and kept.
constexpr int MAX_DEVICES = 64;
std::atomic<void*> scratch_ptr[MAX_DEVICES];

int static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return RAPID_ERR_DEVICE;
    void* ptr = scratch_ptr[dev].load(std::memory_order_acquire);
    if (ptr == nullptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return RAPID_ERR_DEVICE;
        scratch_ptr[dev].store(ptr, std::memory_order_release);   // two threads racing store the same address
    }
    *out = ptr;
    return RAPID_OK;
}

}  // namespace

extern "C" {

int rapid_attn_dense(const void* q, const void* k, const void* v, void* o,
                     int B, int H, int N, int D, int kv_len, float scale,
                     void* workspace, size_t workspace_bytes, void* stream)
{
    (void)workspace; (void)workspace_bytes;
    const int rc = check_common(q, k, v, o, B, H, N, D, kv_len);
    if (rc != RAPID_OK) return rc;
    return run_dense(contiguous_problem(q, k, v, o, B, H, N, D, kv_len, scale), stream);
}

int rapid_attn_block_sparse(const void* q, const void* k, const void* v, void* o,
                            int B, int H, int N, int D, int block,
                            const unsigned char* mask, int kv_len, float scale,
                            void* workspace, size_t workspace_bytes, void* stream)
{
    if (!mask) return RAPID_ERR_NULL;
    const int rc = check_common(q, k, v, o, B, H, N, D, kv_len);
    if (rc != RAPID_OK) return rc;
    if (block != 64 && block != 128) return RAPID_ERR_UNSUPPORTED;
    if (N % block != 0) return RAPID_ERR_SHAPE;
    return run_sparse(contiguous_problem(q, k, v, o, B, H, N, D, kv_len, scale), block, mask, workspace,
                      workspace_bytes, stream);
}

int rapid_attn_joint(const rapid_attn_segment* segments, int n_segments, int B, int H, int D,
                     int block, const unsigned char* mask, int kv_len, const int* kv_lens, float scale,
                     void* workspace, size_t workspace_bytes, void* stream)
{
    Problem pr;
    const int rc = joint_problem(segments, n_segments, B, H, D, block, mask != nullptr, kv_len, kv_lens, scale, pr);
    if (rc != RAPID_OK) return rc;
    if (!mask) return run_dense(pr, stream);
    return run_sparse(pr, block, mask, workspace, workspace_bytes, stream);
}

// Selection and attention in one call: the selection kernels write counts and kept lists where the
// attention's own compaction would have put them; the block means go behind the attention workspace.
int rapid_attn_joint_select(const rapid_attn_segment* segments, int n_segments, int B, int H, int D, int block,
                            int kv_len, const int* kv_lens, int text_start, float tau, float scale,
                            unsigned char* mask_out, void* workspace, size_t workspace_bytes, void* stream)
{
    Problem pr;
    const int rc = joint_problem(segments, n_segments, B, H, D, block, true, kv_len, kv_lens, scale, pr);
    if (rc != RAPID_OK) return rc;
    const int nb = (pr.N + block - 1) / block;
    if ((long long)B * H * nb > 0x7fffffffLL / 16) return RAPID_ERR_SHAPE;
    const WorkspaceLayout w = workspace_layout(B, H, nb, D, block);
    const size_t means = rapid_internal::select_scratch_bytes(B, H, nb, D);
    if (!workspace || workspace_bytes < w.total + means) return RAPID_ERR_WORKSPACE;
    if (!aligned16(workspace)) return RAPID_ERR_ALIGN;
    char* ws = (char*)workspace;
    const int rs = rapid_internal::select_to_lists(segments, n_segments, B, H, D, block, kv_len, kv_lens, text_start, tau,
                                                   scale, mask_out, (int32_t*)(ws + w.counts_off),
                                                   (int32_t*)(ws + w.index_off), ws + w.total, means, stream);
    if (rs != RAPID_OK) return rs;
    return run_sparse(pr, block, nullptr, workspace, w.total, stream);
}

size_t rapid_attn_joint_select_workspace_bytes(int B, int H, int N, int D, int block)
{
    const size_t attn = rapid_attn_joint_workspace_bytes(B, H, N, D, block);
    if (attn == 0 || (N + block - 1) / block > 2048) return 0;
    return attn + rapid_internal::select_scratch_bytes(B, H, (N + block - 1) / block, D);
}

int rapid_attn_block_sparse_static(const void* q, const void* k, const void* v, void* o,
                                   int B, int H, int N, int D, int block,
                                   const unsigned char* mask, int kv_len, float scale, void* stream)
{
    if (!mask) return RAPID_ERR_NULL;
    const int rc = check_common(q, k, v, o, B, H, N, D, kv_len);
    if (rc != RAPID_OK) return rc;
    if (block != 64 && block != 128) return RAPID_ERR_UNSUPPORTED;
    if (N % block != 0) return RAPID_ERR_SHAPE;
    const int nb = N / block;
    if ((long long)B * H * nb > 0x7fffffffLL / 16) return RAPID_ERR_SHAPE;
    // as many partial-result slots as fit next to the lists (fewer slots: fewer items are cut)
    const WorkspaceLayout none = workspace_layout(B, H, nb, D, block, 0);
    if (none.total > (size_t)RAPID_ATTN_STATIC_SCRATCH_BYTES) return RAPID_ERR_WORKSPACE;
    int slots = -1;
    if (workspace_layout(B, H, nb, D, block).total > (size_t)RAPID_ATTN_STATIC_SCRATCH_BYTES) {
        const size_t per_slot = XCDS * ((D == 64 ? PartialSlot<64>::BYTES : PartialSlot<128>::BYTES) + sizeof(PlanRec) + 4);
        slots = (int)(((size_t)RAPID_ATTN_STATIC_SCRATCH_BYTES - none.total) / per_slot);
        while (slots > 0 && workspace_layout(B, H, nb, D, block, slots).total > (size_t)RAPID_ATTN_STATIC_SCRATCH_BYTES) --slots;
    }
    void* ws = nullptr;
    const int rs = static_scratch(&ws);
    if (rs != RAPID_OK) return rs;
    return run_sparse(contiguous_problem(q, k, v, o, B, H, N, D, kv_len, scale), block, mask, ws,
                      (size_t)RAPID_ATTN_STATIC_SCRATCH_BYTES, stream, slots);
}

size_t rapid_attn_joint_workspace_bytes(int B, int H, int N, int D, int block)
{
    if (B <= 0 || H <= 0 || N <= 0 || N > (1 << 22)) return 0;
    if (D != 64 && D != 128) return 0;
    if (block != 64 && block != 128) return 0;
    const int nb = (N + block - 1) / block;
    if ((long long)B * H * nb > 0x7fffffffLL / 16) return 0;
    return workspace_layout(B, H, nb, D, block).total;
}

size_t rapid_attn_workspace_bytes(int B, int H, int N, int D, int block)
{
    if (B <= 0 || H <= 0 || N <= 0) return 0;
    if (D != 64 && D != 128) return 0;
    if (block != 64 && block != 128) return 0;
    if (N % block != 0 || N > (1 << 22)) return 0;
    if ((long long)B * H * (N / block) > 0x7fffffffLL / 16) return 0;
    return workspace_layout(B, H, N / block, D, block).total;
}

const char* rapid_attn_status_string(int status)
{
    switch (status) {
        case RAPID_OK: return "ok";
        case RAPID_ERR_NULL: return "a required pointer is NULL";
        case RAPID_ERR_SHAPE: return "invalid shape: need B,H,N > 0, 1 <= kv_len <= N, N % block == 0";
        case RAPID_ERR_UNSUPPORTED: return "unsupported: D must be 64 or 128, block must be 64 or 128";
        case RAPID_ERR_ALIGN: return "q/k/v/o/workspace must be 16-byte aligned";
        case RAPID_ERR_WORKSPACE: return "workspace is NULL or smaller than rapid_attn_workspace_bytes()";
        case RAPID_ERR_DEVICE: return "HIP runtime refused the launch";
        case RAPID_ERR_ALIAS: return "o overlaps q, k or v";
        default: return "unknown status";
    }
}

int rapid_attn_version(void) { return RAPID_ATTN_VERSION; }

}  // extern "C"
