// Block-sparse attention backward with the selection held fixed (gfx950).
//
// With P the attention weights of the forward pass (recomputed from lse),
//   delta_l = sum_d dO_l[d] O_l[d]
//   dV_t    = sum_l P_lt dO_l
//   dP_lt   = dO_l . v_t,   dS_lt = P_lt (dP_lt - delta_l)
//   dQ_l    = scale sum_t dS_lt k_t,   dK_t = scale sum_l dS_lt q_l
// where (l, t) runs over the pairs the forward pass connects: t in the query's
// own block or in one of its selected blocks.  No gradient flows through the
// top-n choice (Appendix, kernel design paragraph: the backward pass walks, for
// every key/value block, the query blocks connected to it).
//
// Here: the preparation that both backward paths share (delta, the base-2
// log-sum-exps, the reverse map of the selection) and the general-shape kernels on
// the matrix cores (fp32 and bf16, head dim 32, 64 or 128, any tile of up to 1024
// tokens), with the tiles, products and precision of the general forward: the
// rows of the other side are walked as one flat sequence (bsa_flat_rows.h).
//   bwd_generic_dq    a wavefront owns 32 query rows (fp32: 16), walks the attended keys:
//                     S^T = K Q^T and dP^T = V dO^T (a lane holds one query: lse
//                     and delta are scalars of the lane, -delta is the accumulator
//                     that dP^T starts from), dQ^T += K^T dS^T.
//   bwd_generic_dkdv  a wavefront owns 32 (16) rows of a key block, walks the rows of
//                     the query blocks connected to it: S = Q K^T, dP = dO V^T,
//                     dV^T += dO^T P, dK^T += Q^T dS.  The blocks are listed in
//                     ascending order per query head, heads of a group ascending:
//                     the summation order is fixed, there are no floating-point
//                     atomics and results are the same from run to run.
// Launches of few wavefronts split the walk over groups of them (see dkdv_split).
// Measured against the vector-ALU kernels that they replace (a row per four lanes,
// the other side's rows broadcast from LDS): 1.5 degree grid, batch 2, 8 heads,
// head dim 64, bf16, tiles of 10 x 10, 9 blocks: dQ 2.76 -> 0.33 ms, dK and dV
// 4.38 -> 0.57 ms; fp32, batch 1, tiles of 8 x 8: dQ 0.81 -> 0.51 ms, dK and dV 1.55
// -> 1.37 ms (0.97 since the key blocks are ordered).  fp32 with 16-row wavefronts
// instead of 32: dQ 0.48 -> 0.45 ms, dK and dV 0.88 -> 0.67.  delta: 233 -> 21 us and 113 -> 20 us (one thread walked a row).
#include "bsa_device.h"
#include "bsa_flat_rows.h"
#include "bsa_launch.h"
#include "bsa_mfma_common.h"

#include <type_traits>

namespace bsa {

constexpr float kLog2e = 1.4426950408889634f;

// delta_l = dO_l . O_l and lse_l * log2(e).  A row is read by LPR adjacent lanes,
// 16 bytes each, so a wavefront's loads cover whole lines; the partial dot products
// are summed inside the lane group with DPP steps (32 lanes, fp32 rows of 128
// channels: one more exchange).
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(
                   __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

__device__ __forceinline__ float dot16(const uint16_t* a_row, const uint16_t* b_row)
{
    const uint4 a = *(const uint4*)a_row, b = *(const uint4*)b_row;
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
    float acc = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        acc = fmaf(__uint_as_float(aw[e] << 16), __uint_as_float(bw[e] << 16), acc);
        acc = fmaf(__uint_as_float(aw[e] & 0xffff0000u), __uint_as_float(bw[e] & 0xffff0000u),
                   acc);
    }
    return acc;
}
__device__ __forceinline__ float dot16(const float* a_row, const float* b_row)
{
    const float4 a = *(const float4*)a_row, b = *(const float4*)b_row;
    return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x)));
}

template <typename T, int D>
__device__ __forceinline__ void prep_rows(const T* __restrict__ out, const T* __restrict__ dout,
                                          const float* __restrict__ lse, float* __restrict__ delta,
                                          float* __restrict__ lse2, int64_t rows, uint32_t wg)
{
    constexpr int VEC = 16 / (int)sizeof(T), LPR = D / VEC;      // 4, 8, 16 or 32 lanes per row
    const int sub = threadIdx.x % LPR;
    int64_t row = ((int64_t)wg * blockDim.x + threadIdx.x) / LPR;
    const bool valid = row < rows;
    if (!valid) row = rows - 1;                     // keep the lane group whole for the sums
    float acc = dot16(out + row * D + VEC * sub, dout + row * D + VEC * sub);
    acc = dpp_add<0xB1>(acc);                       // quad_perm [1,0,3,2]
    acc = dpp_add<0x4E>(acc);                       // quad_perm [2,3,0,1]
    if (LPR >= 8) acc = dpp_add<0x141>(acc);        // row_half_mirror: 8 lanes
    if (LPR >= 16) acc = dpp_add<0x140>(acc);       // row_mirror: 16 lanes
    if (LPR == 32) acc += __shfl_xor(acc, 16);
    if (valid && sub == 0) {
        delta[row] = acc;
        lse2[row] = lse[row] * kLog2e;
    }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void bwd_prep_kernel(const T* __restrict__ out,
                                                       const T* __restrict__ dout,
                                                       const float* __restrict__ lse,
                                                       float* __restrict__ delta,
                                                       float* __restrict__ lse2, int64_t rows)
{
    prep_rows<T, D>(out, dout, lse, delta, lse2, rows, blockIdx.x);
}

// The reverse map of the selection ("the query blocks connected to a key/value
// block", Appendix, kernel design paragraph) as a bit matrix: bit i % 32 of word
// [query slice][i / 32][key block j] says that query block i attends to block j.
// A dK/dV workgroup reads its bits instead of scanning all m * n entries of the
// slice, and walking the set bits upwards is the fixed summation order.
// One workgroup per (query slice, 32 query blocks) collects its words in LDS (kMapCols
// key blocks at a time) and stores them whole: nothing has to be cleared first and
// no atomic leaves the CU (1.5 degree grid, batch 12, 16 heads, n = 16: 64 -> 8 us
// against one thread per row setting bits in global memory).
constexpr int kMapCols = 8192;

__device__ __forceinline__ void connect_words(const int32_t* __restrict__ sel_idx,
                                              uint32_t* __restrict__ conn, const Geom& g, int words,
                                              uint32_t wg)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t col_s[];   // [min(m, kMapCols)]
    const int m = g.n_blocks, n = g.n_select;
    const int64_t bh_idx = wg / (uint32_t)words;
    const int w = (int)(wg - (uint32_t)bh_idx * (uint32_t)words);
    const int rows = min(32, m - 32 * w);
    const int32_t* sel = sel_idx + (bh_idx * m + 32 * w) * n;
    uint32_t* dst = conn + (bh_idx * words + w) * m;
    for (int j0 = 0; j0 < m; j0 += kMapCols) {
        const int cols = min(kMapCols, m - j0);
        for (int c = threadIdx.x; c < cols; c += blockDim.x) col_s[c] = 0u;
        __syncthreads();
        for (int e = threadIdx.x; e < rows * n; e += blockDim.x) {
            const int j = sel[e] - j0;
            if ((unsigned)j < (unsigned)cols) atomicOr(&col_s[j], 1u << (e / n));
        }
        // the own block, unless only the lists count
        const int own = 32 * w + (int)threadIdx.x - j0;
        if (!g.list_only && (int)threadIdx.x < rows && (unsigned)own < (unsigned)cols)
            atomicOr(&col_s[own], 1u << threadIdx.x);
        __syncthreads();
        for (int c = threadIdx.x; c < cols; c += blockDim.x) dst[j0 + c] = col_s[c];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void bwd_connect_kernel(const int32_t* __restrict__ sel_idx,
                                                          uint32_t* __restrict__ conn, Geom g,
                                                          int words)
{
    connect_words(sel_idx, conn, g, words, blockIdx.x);
}

// The map and delta in one launch, the map's workgroups first: both are short, read nothing
// of each other, and a launch of its own costs a small backward 4.5 us.
template <typename T, int D>
__global__ __launch_bounds__(256) void bwd_prep_connect_kernel(
    const T* __restrict__ out, const T* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ delta, float* __restrict__ lse2, int64_t rows,
    const int32_t* __restrict__ sel_idx, uint32_t* __restrict__ conn, Geom g, int words,
    uint32_t n_connect)
{
    if (blockIdx.x < n_connect)
        connect_words(sel_idx, conn, g, words, blockIdx.x);
    else
        prep_rows<T, D>(out, dout, lse, delta, lse2, rows, blockIdx.x - n_connect);
}

// The order in which the key blocks of a key/value slice are worked on: those with
// many connected query blocks first.  The number of connections is far from even
// (on smooth fields the most popular block has 4 to 7 times the mean), and a
// workgroup that walks the longest list alone at the end of a launch keeps the
// rest of the chip waiting.  Five classes, each in ascending block order:
// neighbours, which share connected blocks, stay together.  dK/dV kernels, 1.5
// degree grid: fp32, 8 slices, 9 blocks: 1.37 -> 0.97 ms (the longest of 3,600 lists
// is 61 blocks, 0.5 ms of work); bf16, 48 key/value slices of 4 heads: 4.13 ->
// 3.96 ms.
constexpr int kClasses = 5;

// Class of key block j of the slice whose query slices' map words start at base
// (`all_words` columns of m words).  What bounds it is the latency of the reads.
__device__ __forceinline__ int connection_class(const uint32_t* __restrict__ base, int m, int j,
                                                int all_words, int mean)
{
    constexpr int BATCH = 16;
    const uint32_t* at = base + j;
    int deg = 0, w = 0;
    for (; w + BATCH <= all_words; w += BATCH, at += (int64_t)BATCH * m) {
        uint32_t x[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) x[u] = at[(int64_t)u * m];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) deg += __builtin_popcount(x[u]);
    }
    for (; w < all_words; ++w, at += m) deg += __builtin_popcount(*at);
    return deg >= 4 * mean ? 0 : deg >= 3 * mean ? 1 : deg >= 2 * mean ? 2
           : 2 * deg >= 3 * mean ? 3 : 4;
}

// First query slice of key/value slice u.
__device__ __forceinline__ int64_t first_query_slice(const Geom& g, int64_t u)
{
    const int64_t kv_heads = g.heads / g.kv_group;
    return (u / kv_heads) * g.heads + (u % kv_heads) * g.kv_group;
}

// The classes of all key blocks by the whole chip, for maps that are too large to be
// read by one workgroup per slice; see launch_order.
__global__ __launch_bounds__(256) void bwd_class_kernel(const uint32_t* __restrict__ conn,
                                                        uint8_t* __restrict__ classes, Geom g,
                                                        int words, uint32_t chunks)
{
    const int m = g.n_blocks;
    const int64_t unit = blockIdx.x / chunks;
    const int j = (int)((blockIdx.x % chunks) * 256 + threadIdx.x);
    if (j >= m) return;
    classes[unit * m + j] = (uint8_t)connection_class(
        conn + first_query_slice(g, unit) * words * (int64_t)m, m, j, g.kv_group * words,
        g.kv_group * (g.n_select + 1 - g.list_only));
}

// One workgroup per key/value slice.  classes: from bwd_class_kernel, or null, then the
// workgroup has a thread per key block.
__global__ __launch_bounds__(1024) void bwd_order_kernel(const uint32_t* __restrict__ conn,
                                                         const uint8_t* __restrict__ classes,
                                                         int32_t* __restrict__ order, Geom g,
                                                         int words)
{
    __shared__ int count_s[16][kClasses], start_s[kClasses];
    const int m = g.n_blocks, threads = blockDim.x, waves = threads >> 6;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t unit = blockIdx.x;
    order += unit * m;
    if (classes) classes += unit * m;
    int first_class = kClasses;                      // of block threadIdx.x
    if ((int)threadIdx.x < m)
        first_class = classes ? classes[threadIdx.x]
                              : connection_class(conn + first_query_slice(g, unit) * words * (int64_t)m,
                                                 m, threadIdx.x, g.kv_group * words,
                                                 g.kv_group * (g.n_select + 1 - g.list_only));
    // sizes of the classes
    int mine[kClasses];
#pragma unroll
    for (int c = 0; c < kClasses; ++c) mine[c] = first_class == c ? 1 : 0;
    for (int j = threadIdx.x + threads; j < m; j += threads) {
        const int cls = classes[j];
#pragma unroll
        for (int c = 0; c < kClasses; ++c) mine[c] += cls == c ? 1 : 0;
    }
#pragma unroll
    for (int c = 0; c < kClasses; ++c) {
        for (int off = 32; off >= 1; off >>= 1) mine[c] += __shfl_xor(mine[c], off);
        if (lane == 0) count_s[wave][c] = mine[c];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int at = 0;
        for (int c = 0; c < kClasses; ++c) {
            start_s[c] = at;
            for (int w = 0; w < waves; ++w) at += count_s[w][c];
        }
    }
    __syncthreads();
    // a block per thread at a time, in ascending order inside each class
    for (int j0 = 0; j0 < m; j0 += threads) {
        const int j = j0 + (int)threadIdx.x;
        const int cls = j0 == 0 ? first_class : j < m ? classes[j] : kClasses;
        int before = 0;
#pragma unroll
        for (int c = 0; c < kClasses; ++c) {
            const uint64_t mask = __builtin_amdgcn_ballot_w64(cls == c);
            if (cls == c) before = __builtin_popcountll(mask & ((1ull << lane) - 1));
            if (lane == 0) count_s[wave][c] = __builtin_popcountll(mask);
        }
        __syncthreads();
        if (j < m) {
            int at = start_s[cls] + before;
            for (int w = 0; w < wave; ++w) at += count_s[w][cls];
            order[at] = j;
        }
        __syncthreads();
        if (threadIdx.x < kClasses)
            for (int w = 0; w < waves; ++w) start_s[threadIdx.x] += count_s[w][threadIdx.x];
        __syncthreads();
    }
}

static hipError_t launch_connect(const int32_t* sel_idx, uint32_t* conn, const Geom& g, int64_t BH,
                                 hipStream_t stream)
{
    const int m = g.n_blocks, words = (m + 31) >> 5;
    const int cols = m < kMapCols ? m : kMapCols;
    const int64_t map = (int64_t)words * m;          // words per query slice
    return launch_slices(BH, 256 * (int64_t)words, [&](int64_t first, int64_t slices) {
        bwd_connect_kernel<<<dim3((unsigned)(slices * words)), dim3(256),
                             sizeof(uint32_t) * (size_t)cols, stream>>>(
            sel_idx + first * m * g.n_select, conn + first * map, g, words);
        return hipGetLastError();
    });
}

static hipError_t launch_order(const uint32_t* conn, int32_t* order, const Geom& g, int64_t BH,
                               hipStream_t stream)
{
    const int m = g.n_blocks, words = (m + 31) >> 5;
    const int64_t map = (int64_t)words * m;
    hipError_t e = hipSuccess;
    // A slice's map of up to 1,024 blocks and 64 words each is read where the order is
    // made, a larger one by a launch of its own: 450 blocks with 60 words 9.9 us, in two
    // launches 6.9 + 4.9; 1,024 with 128 8.0 + 5.0 us, 4,050 with 127 9.7 + 10.8 us (one
    // workgroup per slice, counting twice: 93 and 205 us; the training pass of one slice
    // of 16,200 blocks 8.9 -> 4.3 ms).
    const int64_t BKV = BH / g.kv_group;
    uint8_t* classes = nullptr;
    if (m > 1024 || g.kv_group * words > 64) {
        const uint32_t chunks = (uint32_t)(m + 255) / 256;
        classes = (uint8_t*)(order + BKV * m);
        e = launch_slices(BKV, 256 * (int64_t)chunks, [&](int64_t first, int64_t slices) {
            bwd_class_kernel<<<dim3((unsigned)(slices * chunks)), dim3(256), 0, stream>>>(
                conn + first * g.kv_group * map, classes + first * m, g, words, chunks);
            return hipGetLastError();
        });
        if (e != hipSuccess) return e;
    }
    const int threads = m >= 1024 ? 1024 : (m + 63) / 64 * 64;
    return launch_slices(BKV, threads, [&](int64_t first, int64_t slices) {
        bwd_order_kernel<<<dim3((unsigned)slices), dim3(threads), 0, stream>>>(
            conn + first * g.kv_group * map, classes ? classes + first * m : nullptr,
            order + first * m, g, words);
        return hipGetLastError();
    });
}

template <typename T, int D>
static hipError_t launch_prep_t(const void* out, const void* dout, const float* lse, float* delta,
                                float* lse2, int64_t rows, const int32_t* sel_idx, uint32_t* conn,
                                const Geom& g, int64_t BH, hipStream_t stream)
{
    constexpr int LPR = D * (int)sizeof(T) / 16, RPW = 256 / LPR;     // rows per workgroup
    const int64_t wgs = (rows + RPW - 1) / RPW;
    // together with the map where its LDS leaves the rows' workgroups alone and one launch
    // holds both
    const int m = g.n_blocks, words = (m + 31) >> 5;
    const int64_t n_connect = BH * words;
    if (m <= 1024 && (wgs + n_connect) * 256 < (int64_t)1 << 32) {
        bwd_prep_connect_kernel<T, D><<<dim3((unsigned)(wgs + n_connect)), dim3(256),
                                        sizeof(uint32_t) * (size_t)m, stream>>>(
            (const T*)out, (const T*)dout, lse, delta, lse2, rows, sel_idx, conn, g, words,
            (uint32_t)n_connect);
        return hipGetLastError();
    }
    const hipError_t e = launch_slices(wgs, 256, [&](int64_t first, int64_t count) {
        const int64_t row = first * RPW;
        bwd_prep_kernel<T, D><<<dim3((unsigned)count), dim3(256), 0, stream>>>(
            (const T*)out + row * D, (const T*)dout + row * D, lse + row, delta + row, lse2 + row,
            rows - row < count * RPW ? rows - row : count * RPW);
        return hipGetLastError();
    });
    return e != hipSuccess ? e : launch_connect(sel_idx, conn, g, BH, stream);
}

hipError_t launch_bwd_prepare(bool is_bf16, const void* out, const void* dout, const float* lse,
                              float* delta, float* lse2, const int32_t* sel_idx, uint32_t* conn,
                              int32_t* order, const Geom& g, int D, int64_t BH, hipStream_t stream)
{
    hipError_t e = hipErrorInvalidValue;
    if (!lse) e = launch_connect(sel_idx, conn, g, BH, stream);
#define BSA_CASE(DD)                                                                              \
    else if (D == DD)                                                                             \
        e = is_bf16 ? launch_prep_t<uint16_t, DD>(out, dout, lse, delta, lse2, BH * g.n_tokens,   \
                                                  sel_idx, conn, g, BH, stream)                   \
                    : launch_prep_t<float, DD>(out, dout, lse, delta, lse2, BH * g.n_tokens,      \
                                               sel_idx, conn, g, BH, stream);
    BSA_CASE(32)
    BSA_CASE(64)
    BSA_CASE(128)
#undef BSA_CASE
    return e != hipSuccess || !order ? e : launch_order(conn, order, g, BH, stream);
}

// ---------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------
// Launch bounds (wavefronts per SIMD as the registers allow, 32-row bf16 against 16-row
// fp32 wavefronts) and the most wavefronts of a workgroup: 4 where three of them share a
// SIMD (workgroups of 8 would leave it two), so that larger fp32 blocks are split.  fp32,
// blocks of 128, head dim 64, 8 slices: training pass 2.90 ms with workgroups of 8, 2.65
// with 4; head dim 128, 5.58 ms with one wavefront per SIMD in dK/dV, 5.29 with two (27
// registers spill outside of the tile loop), but 2.63 against 3.52 where two wavefronts
// gather, which then reload inside the loop.
template <typename T, int D> struct BwdLimits {
    static constexpr bool WIDE = sizeof(T) == 2 && D == 128;
    static constexpr int MAX_WAVES = WIDE || sizeof(T) == 4 ? 4 : 8;
    static constexpr int PER_SIMD = WIDE ? 1 : sizeof(T) == 4 && D < 128 ? 3 : 2;
};
// The bounds of one form: SPLIT groups of NL wavefronts; unsplit (SPLIT 1) NL wavefronts that
// gather: 1 of 1, 2 of up to 3 (3: dQ of head dim 128 has a form for exactly three), 4 of up to
// MAX_WAVES.  Wavefronts per SIMD that the registers must leave room for:
//   * unsplit: what BwdLimits says from four wavefronts on.  A lone wavefront may take them all: its
//     workgroups fill a CU's LDS before its SIMDs.  Two or three in dQ as from four on, at head dim
//     128 dQ of three and more 2 (two workgroups of three fit a CU and share its SIMDs); in dK/dV,
//     with twice the accumulators, 2 below head dim 128 and 1 there.
//   * split: as many workgroups as LDS holds.  dQ 1 (it is split only where they are few); dK/dV 2
//     where LDS holds eight wavefronts: head dim 32, bf16 of 64 (four single wavefronts spill 4
//     registers outside of the tile loop) and fp32 of 64 in pairs, else 1.
template <typename T, int D, int NL, int SPLIT> struct BwdBounds {
    using L = BwdLimits<T, D>;
    static constexpr bool F32 = sizeof(T) == 4;
    static constexpr int THREADS = SPLIT > 1 ? 64 * SPLIT * NL
                                   : NL == 4 ? 64 * L::MAX_WAVES : NL == 1 ? 64 : 192;
    static constexpr int DQ = SPLIT > 1 || NL == 1 ? 1 : D == 128 && NL > 2 ? 2 : L::PER_SIMD;
    static constexpr int SPLIT_DKDV =
        D == 32 || (D == 64 && (!F32 || (NL == 2 && SPLIT == 2))) ? 2 : 1;
    static constexpr int DKDV = SPLIT > 1 ? SPLIT_DKDV
                                : NL == 4 ? L::PER_SIMD : NL == 2 && D < 128 ? 2 : 1;
};

// Launches that leave most of the chip idle, or wait for the longest list of a few key
// blocks: SPLIT groups of NL wavefronts own the same rows, and each takes 32 rows (bf16 in
// two groups: of the same 64) of a tile that all of them gather.  The first group adds up
// what the others have at the end, in the order of the groups.
template <typename T, int D, int SPLIT>
using SplitTile = FlatTile<T, D, (SPLIT > 1 ? 32 * SPLIT : FlatTile<T, D>::KT)>;

// Adds `count` accumulators of groups 1 .. SPLIT - 1 to those of group 0, lane by lane,
// through the tiles' memory.  All wavefronts call it; false: not group 0.
template <int SPLIT, int NL, int COUNT, int BYTES, class V>
__device__ __forceinline__ bool add_groups(unsigned char* lds_a, unsigned char* lds_b, int group,
                                           int wave, int lane, V (&acc)[COUNT])
{
    constexpr int PER = (int)sizeof(V) / 4, HALF = BYTES / 256;    // values per array and lane
    static_assert((SPLIT - 1) * NL * COUNT * PER <= 2 * HALF, "fits the tiles");
    auto place = [&](int from, int value) -> float* {
        const int at = ((from - 1) * NL + wave) * COUNT * PER + value;
        return (at < HALF ? (float*)lds_a + at * 64 : (float*)lds_b + (at - HALF) * 64) + lane;
    };
    __syncthreads();
    if (group > 0) {
#pragma unroll
        for (int c = 0; c < COUNT; ++c)
#pragma unroll
            for (int r = 0; r < PER; ++r) *place(group, c * PER + r) = acc[c][r];
    }
    __syncthreads();
    if (group > 0) return false;
    for (int from = 1; from < SPLIT; ++from)
#pragma unroll
        for (int c = 0; c < COUNT; ++c)
#pragma unroll
            for (int r = 0; r < PER; ++r) acc[c][r] += *place(from, c * PER + r);
    return true;
}

template <typename T, int D, int NL, int SPLIT, bool MIXED = false>
__global__ __launch_bounds__((BwdBounds<T, D, NL, SPLIT>::THREADS), (BwdBounds<T, D, NL, SPLIT>::DQ))
void bwd_generic_dq(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                    const T* __restrict__ dout, const float* __restrict__ lse2,
                    const float* __restrict__ delta, const int32_t* __restrict__ sel_idx,
                    T* __restrict__ dq, Geom g, uint32_t n_units, int row_chunks, int chunk_rows)
{
    using Tile = SplitTile<T, D, SPLIT>;
    constexpr int KT = Tile::KT, LOADERS = SPLIT > 1 ? SPLIT * NL : NL == 3 ? 2 : NL;
    constexpr int PIECES = KT / 32 / SPLIT;          // of a tile, for each group
    __shared__ __attribute__((aligned(1024))) unsigned char k_lds[2][Tile::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_lds[2][Tile::TILE_BYTES];
    extern __shared__ __attribute__((aligned(16))) uint32_t tables_s[];

    const int lane = threadIdx.x & 63;
    const int wg_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = SPLIT == 1 ? 0 : wg_wave / NL, wave = wg_wave - group * NL;
    const int b = g.block_tokens;

    int item;
    int64_t bh_idx;
    map_workgroup(g, blockIdx.x, (uint32_t)row_chunks, n_units, bh_idx, item);
    const int i = item / row_chunks;
    const int row0 = (item - i * row_chunks) * chunk_rows;
    const int64_t base = bh_idx * g.n_tokens * D;
    const int64_t kv_base = kv_slice_of(g, bh_idx) * g.n_tokens * D;

    AttendedKeys<T, D, LOADERS, 1, Tile> keys;
    keys.init(g, sel_idx, bh_idx, i, tables_s, lane, wg_wave);

    const int first_row = row0 + WaveTile<T>::ROWS * wave, end_row = min(b, row0 + chunk_rows);

    with_rows<T, MIXED>(end_row - first_row, [&](auto piece_key) {
    using K = typename decltype(piece_key)::type;
    using W = WaveTile<K>;
    const int col = lane & (W::ROWS - 1), part = lane / W::ROWS;
    TileReader<K, D> rd;
    rd.init(lane);
    const int tau_q = first_row + col;
    const bool valid = tau_q < end_row;
    const int64_t q_tok = token_of(g, i, valid ? tau_q : 0);
    typename RowPieces<K, D>::type qf[RowPieces<K, D>::N], dof[RowPieces<K, D>::N];
#pragma unroll
    for (int s = 0; s < RowPieces<K, D>::N; ++s) {
        load_row<K>(q + base + q_tok * D, qf[s], s, part);
        load_row<K>(dout + base + q_tok * D, dof[s], s, part);
    }
    const float neg_l2 = -lse2[bh_idx * g.n_tokens + q_tok];
    const float neg_delta = -delta[bh_idx * g.n_tokens + q_tok];
    const float c2 = g.scale * kLog2e;
    Column<K, D> acc;
    clear_column<K, D>(acc);
    const typename W::vec dp0 = constant_tile<K>(neg_delta);

    __syncthreads();                                 // tables
    const int64_t slice_bytes = g.n_tokens * Tile::ROW_BYTES;
    const RowSource ks(k + kv_base, slice_bytes), vs(v + kv_base, slice_bytes);
    const uint32_t k_dst = lds_address(k_lds), v_dst = lds_address(v_lds);
    if (wg_wave < LOADERS) {
        keys.look_up();
        keys.gather_next(ks, vs, k_dst, v_dst);
    }
    for (int c = 0; c < keys.tiles; ++c) {
        // tile c has landed and everyone is done with the other buffer
        wait_gathers();
        __syncthreads();
        const int buf = c & 1, other = (buf ^ 1) * Tile::TILE_BYTES;
        if (wg_wave < LOADERS && c + 1 < keys.tiles) keys.gather_next(ks, vs, k_dst + other, v_dst + other);
#pragma unroll
        for (int hh = 0; hh < PIECES; ++hh) {
            constexpr int HALF = 32 * Tile::ROW_BYTES;
            const uint32_t at = (uint32_t)(buf * Tile::TILE_BYTES + group * PIECES * HALF);
            const uint32_t kt = k_dst + at, vt = v_dst + at;
            const int left = keys.total - (KT * c + 32 * (group * PIECES + hh));
            if (left <= 0) break;
            typename W::vec s = constant_tile<K>(0.0f), dp = dp0;
            dot_tiles<false, K, D>(rd, kt, vt, hh * HALF, qf, dof, s, dp);
            ColumnPieces<K, D> k0;
            read_columns(rd, kt, hh * HALF, 0, k0);
            if (left < 32)
#pragma unroll
                for (int r = 0; r < W::NR; ++r)
                    if (past_end<K>(r, part, left)) s[r] = -INFINITY;
#pragma unroll
            for (int r = 0; r < W::NR; ++r) dp[r] *= __builtin_amdgcn_exp2f(fmaf(s[r], c2, neg_l2));
            weighted_rows(rd, kt, hh * HALF, k0, dp, acc);
        }
    }

    if constexpr (SPLIT > 1)
        if (!add_groups<SPLIT, NL, sizeof(acc.a) / sizeof(acc.a[0]), 2 * Tile::TILE_BYTES>(
                k_lds[0], v_lds[0], group, wave, lane, acc.a))
            return;
    if (valid) {
        const float inv_b = 1.0f / (float)b;
        const float* extra = g.add_dq ? g.add_dq + (bh_idx * g.n_blocks + i) * D : nullptr;
        store_column<D>(dq + base + q_tok * D, acc, g.scale, extra, inv_b, part);
    }
    });
}

// ---------------------------------------------------------------------------
// dK, dV
// ---------------------------------------------------------------------------
// The list of connected query blocks holds up to kConnCap of them; it is filled
// 1024 blocks (32 words of the reverse map) at a time while it has room for all of
// them, and walked whenever it is full or the map is exhausted.
constexpr int kConnCap = 2048;

template <typename T, int D, int NL, int SPLIT, bool MIXED = false>
__global__ __launch_bounds__((BwdBounds<T, D, NL, SPLIT>::THREADS), (BwdBounds<T, D, NL, SPLIT>::DKDV))
void bwd_generic_dkdv(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                      const T* __restrict__ dout, const float* __restrict__ lse2,
                      const float* __restrict__ delta, const uint32_t* __restrict__ conn,
                      const int32_t* __restrict__ order, T* __restrict__ dk, T* __restrict__ dv, Geom g, uint32_t n_units,
                      int row_chunks, int chunk_rows)
{
    using Tile = SplitTile<T, D, SPLIT>;
    constexpr int KT = Tile::KT, LOADERS = SPLIT > 1 ? SPLIT * NL : NL;
    constexpr int MINE = Tile::SLABS / LOADERS;
    static_assert(Tile::SLABS % LOADERS == 0, "slabs split evenly between the loading wavefronts");
    constexpr int PIECES = KT / 32 / SPLIT;           // of a tile, for each group
    constexpr int LROWS = KT < 64 ? 64 : KT, LWAVES = LROWS / 64;   // lse, delta: loads of 64 rows
    __shared__ __attribute__((aligned(1024))) unsigned char q_lds[2][Tile::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char g_lds[2][Tile::TILE_BYTES];
    __shared__ __attribute__((aligned(256))) float l_lds[2][LROWS];
    __shared__ __attribute__((aligned(256))) float d_lds[2][LROWS];
    __shared__ uint32_t list_s[kConnCap + repeated_entries(KT, 1)];   // first token (in the group's
                                                      // rows) per block, the last one repeated
    __shared__ int state_s[2];                        // blocks listed, words left
    extern __shared__ __attribute__((aligned(16))) uint32_t pos_s[];        // [b]

    const int lane = threadIdx.x & 63;
    const int wg_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = SPLIT == 1 ? 0 : wg_wave / NL, wave = wg_wave - group * NL;
    const int m = g.n_blocks, b = g.block_tokens;
    const int words = (m + 31) >> 5;                  // of a key block's row of the reverse map

    // workgroup -> (key/value slice, key block, row chunk); the query slices that share the
    // key/value slice are consecutive
    uint32_t unit, item;
    map_key_block(g, blockIdx.x, (uint32_t)row_chunks, n_units, unit, item);
    const int place = (int)item / row_chunks;
    const int row0 = ((int)item - place * row_chunks) * chunk_rows;
    const int j = order ? order[(int64_t)unit * m + place] : place;
    const int64_t base = (int64_t)unit * g.n_tokens * D;
    int64_t bh_first;
    {
        const uint32_t kv_heads = (uint32_t)(g.heads / g.kv_group);
        const uint32_t e = unit / kv_heads, a = unit - e * kv_heads;
        bh_first = (int64_t)e * g.heads + (int64_t)a * g.kv_group;
    }
    const int64_t group_rows = g.kv_group * g.n_tokens;
    const RowSource qs(q + bh_first * g.n_tokens * D, group_rows * Tile::ROW_BYTES),
        gs(dout + bh_first * g.n_tokens * D, group_rows * Tile::ROW_BYTES);
    const float* lb = lse2 + bh_first * g.n_tokens;
    const float* db = delta + bh_first * g.n_tokens;
    const i32x4 l_rsrc = buffer_desc(lb, (uint32_t)(group_rows * 4)),
                d_rsrc = buffer_desc(db, (uint32_t)(group_rows * 4));

    fill_position_table(g, pos_s);
    const int first_row = row0 + WaveTile<T>::ROWS * wave, end_row = min(b, row0 + chunk_rows);

    with_rows<T, MIXED>(end_row - first_row, [&](auto piece_key) {
    using K = typename decltype(piece_key)::type;
    using W = WaveTile<K>;
    const int col = lane & (W::ROWS - 1), part = lane / W::ROWS;
    TileReader<K, D> rd;
    rd.init(lane);

    // this wavefront's key rows.  V enters negated: the accumulator that starts
    // from delta then ends as delta - dP without an instruction per element, and
    // dK is stored with the sign turned.
    const int tau_k = first_row + col;
    const bool valid = tau_k < end_row;
    const int64_t k_tok = token_of(g, j, valid ? tau_k : 0);
    typename RowPieces<K, D>::type kf[RowPieces<K, D>::N], vf[RowPieces<K, D>::N];
#pragma unroll
    for (int s = 0; s < RowPieces<K, D>::N; ++s) {
        load_row<K>(k + base + k_tok * D, kf[s], s, part);
        load_row<K>(v + base + k_tok * D, vf[s], s, part);
        vf[s] = negated(vf[s]);
    }
    const float c2 = g.scale * kLog2e;
    Column<K, D> acck, accv;
    clear_column<K, D>(acck);
    clear_column<K, D>(accv);

    const uint32_t q_dst = lds_address(q_lds), g_dst = lds_address(g_lds);
    const uint32_t l_dst = lds_address(l_lds), d_dst = lds_address(d_lds);
    const uint32_t step_q = (uint32_t)(KT / b), step_r = (uint32_t)(KT % b);

    // the map's words of the group's heads, head-major: one flat sequence
    const int all_words = g.kv_group * words;
    int next_word = 0;                                // wavefront 0 only
    for (;;) {
        __syncthreads();                              // the previous list is used up
        if (wg_wave == 0) {
            int count = 0;
            while (next_word < all_words && count <= kConnCap - 1024) {
                const int w = next_word + lane;
                uint32_t bits = 0;
                int gq = 0, wi = 0;
                if (lane < 32 && w < all_words) {
                    gq = w / words;
                    wi = w - gq * words;
                    bits = conn[((bh_first + gq) * words + wi) * m + j];
                }
                const int mine = __builtin_popcount(bits);
                int upto = mine;                      // inclusive prefix sum over the lanes
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int t = __shfl_up(upto, off);
                    upto += lane >= off ? t : 0;
                }
                int at = count + upto - mine;
                while (bits) {
                    const int i = 32 * wi + __builtin_ctz(bits);
                    bits &= bits - 1;
                    list_s[at++] = (uint32_t)gq * (uint32_t)g.n_tokens + block_first_token(g, i);
                }
                count += __builtin_amdgcn_readlane(upto, 63);
                next_word += 32;
            }
            if (lane == 0) {
                state_s[0] = count;
                state_s[1] = next_word < all_words ? 1 : 0;
            }
        }
        __syncthreads();
        const int listed = __builtin_amdgcn_readfirstlane(state_s[0]);
        const bool more = __builtin_amdgcn_readfirstlane(state_s[1]) != 0;
        if (listed == 0) {
            if (!more) break;
            continue;
        }
        // rows past the end of the last tile take rows of the last block
        const int repeats = repeated_entries(KT, b);
        for (int e = threadIdx.x; e < repeats; e += blockDim.x)
            list_s[listed + e] = list_s[listed - 1];
        __syncthreads();
        const int total = listed * b;
        const int tiles = (total + KT - 1) / KT;

        // this lane's rows of a tile (slab wg_wave + LOADERS jj), and for the loads of lse
        // and delta row 64 wg_wave + lane (32 rows: the upper lanes repeat the lower ones;
        // rows of the tile after the last one would lie past the repeated entries)
        FlatRow at[MINE], at_row;
        uint32_t chunk_off[MINE], tok[MINE], tok_row = 0;
#pragma unroll
        for (int jj = 0; jj < MINE; ++jj) {
            const int row = Tile::RPS * (wg_wave + LOADERS * jj) + lane / Tile::LPR;
            at[jj].start(row, b);
            chunk_off[jj] = (uint32_t)Tile::swz(row, lane % Tile::LPR) * 16u;
        }
        if (wg_wave < LWAVES) at_row.start(64 * wg_wave + lane % KT, b);
        auto row_of = [&](const FlatRow& r) -> uint32_t { return list_s[r.blk] + pos_s[r.tau]; };
        // rows of the next tile, looked up a tile before they are used
        auto look_up = [&] {
#pragma unroll
            for (int jj = 0; jj < MINE; ++jj) {
                tok[jj] = row_of(at[jj]);
                at[jj].advance(step_q, step_r, b);
            }
            if (wg_wave < LWAVES) {
                tok_row = row_of(at_row);
                at_row.advance(step_q, step_r, b);
            }
        };
        auto gather_next = [&](int buf) {
            gather_rows<Tile, MINE, LOADERS>(qs, gs, tok, chunk_off, wg_wave,
                                        q_dst + (uint32_t)buf * Tile::TILE_BYTES,
                                        g_dst + (uint32_t)buf * Tile::TILE_BYTES);
            if (wg_wave < LWAVES) {
                const uint32_t to = (uint32_t)(buf * LROWS + 64 * wg_wave) * 4u;
                if (__builtin_expect(!qs.wide, 1)) {
                    load_lds_4(l_rsrc, tok_row * 4u, 0u, l_dst + to);
                    load_lds_4(d_rsrc, tok_row * 4u, 0u, d_dst + to);
                } else {
                    load_lds_4_at(lb + tok_row, l_dst + to);
                    load_lds_4_at(db + tok_row, d_dst + to);
                }
            }
            look_up();
        };
        if (wg_wave < LOADERS) {
            look_up();
            gather_next(0);
        }
        for (int c = 0; c < tiles; ++c) {
            wait_gathers();
            __syncthreads();
            const int buf = c & 1;
            if (wg_wave < LOADERS && c + 1 < tiles) gather_next(buf ^ 1);
#pragma unroll
            for (int hh = 0; hh < PIECES; ++hh) {
                constexpr int HALF = 32 * Tile::ROW_BYTES;
                const uint32_t first = (uint32_t)(buf * Tile::TILE_BYTES + group * PIECES * HALF);
                const uint32_t qt = q_dst + first, gt = g_dst + first;
                const int row = 32 * (group * PIECES + hh), left = total - (KT * c + row);
                if (left <= 0) break;
                typename W::vec p = constant_tile<K>(0.0f), dp;
#pragma unroll
                for (int r4 = 0; r4 < W::NR / 4; ++r4) {
                    const float4 d4 = *(const float4*)(d_lds[buf] + row + W::STEP * r4 + 4 * part);
                    dp[4 * r4] = d4.x; dp[4 * r4 + 1] = d4.y;
                    dp[4 * r4 + 2] = d4.z; dp[4 * r4 + 3] = d4.w;
                }
                dot_tiles<true, K, D>(rd, qt, gt, hh * HALF, kf, vf, p, dp);
                ColumnPieces<K, D> c0;
                read_columns(rd, gt, hh * HALF, 0, c0);
                if (left < 32)
#pragma unroll
                    for (int r = 0; r < W::NR; ++r)
                        if (past_end<K>(r, part, left)) p[r] = -INFINITY;
#pragma unroll
                for (int r4 = 0; r4 < W::NR / 4; ++r4) {
                    const float4 l4 = *(const float4*)(l_lds[buf] + row + W::STEP * r4 + 4 * part);
                    p[4 * r4] = __builtin_amdgcn_exp2f(fmaf(p[4 * r4], c2, -l4.x));
                    p[4 * r4 + 1] = __builtin_amdgcn_exp2f(fmaf(p[4 * r4 + 1], c2, -l4.y));
                    p[4 * r4 + 2] = __builtin_amdgcn_exp2f(fmaf(p[4 * r4 + 2], c2, -l4.z));
                    p[4 * r4 + 3] = __builtin_amdgcn_exp2f(fmaf(p[4 * r4 + 3], c2, -l4.w));
                }
                weighted_rows(rd, gt, hh * HALF, c0, p, accv);
                read_columns(rd, qt, hh * HALF, 0, c0);
#pragma unroll
                for (int r = 0; r < W::NR; ++r) dp[r] *= p[r];
                weighted_rows(rd, qt, hh * HALF, c0, dp, acck);
            }
        }
        if (!more) break;
    }

    if constexpr (SPLIT > 1) {
        constexpr int COUNT = sizeof(acck.a) / sizeof(acck.a[0]);
        typename std::remove_reference<decltype(acck.a[0])>::type both[2 * COUNT];
#pragma unroll
        for (int c = 0; c < COUNT; ++c) {
            both[c] = acck.a[c];
            both[COUNT + c] = accv.a[c];
        }
        if (!add_groups<SPLIT, NL, 2 * COUNT, 2 * Tile::TILE_BYTES>(q_lds[0], g_lds[0], group, wave,
                                                                    lane, both))
            return;
#pragma unroll
        for (int c = 0; c < COUNT; ++c) {
            acck.a[c] = both[c];
            accv.a[c] = both[COUNT + c];
        }
    }
    if (valid) {
        const float inv_b = 1.0f / (float)b;
        const int64_t pooled_row = ((int64_t)unit * m + j) * D;
        store_column<D>(dk + base + k_tok * D, acck, -g.scale,
                           g.add_dk ? g.add_dk + pooled_row : nullptr, inv_b, part);
        store_column<D>(dv + base + k_tok * D, accv, 1.0f,
                           g.add_dv ? g.add_dv + pooled_row : nullptr, inv_b, part);
    }
    });
}

// Row wavefronts of a workgroup at most, and groups that share its list, by the row
// wavefronts of the launch and the rows that one of them walks on average, in pieces of
// 32.  What bounds a launch of few wavefronts is the longest list, walked by wavefronts
// whose SIMDs have nothing else to do: on smooth fields the most popular key block has 4
// to 7 times the mean of dK/dV, and dQ's lists are short chains on an idle chip.  What a
// split costs is two barriers and the sum of the accumulators through LDS (1 to 3 us),
// pairs of row wavefronts that gather for themselves, and at four groups the LDS of a
// tile twice as large.  Whole backward, us, unsplit | pairs of wavefronts, two groups |
// single ones, four groups (slices x blocks x tokens, attended blocks):
//   bf16, head dim 64:   1 x 24 x 130, 13:   152 | 104 | 88     1 x 96 x 130, 13:  198 | 134 | 108
//                        4 x 96 x 80, 13:    156 | 132 | 112    1 x 448 x 130, 13: 329 | 263 | 259
//                        1 x 448 x 255, 4:   292 | 212 | 248    16 x 96 x 255, 4:  600 | 625 | 741
//   bf16, head dim 128:  1 x 96 x 36, 13:    139 | 100 | 84     1 x 448 x 36, 13:  187 | 131 | 143
//                        4 x 448 x 36, 13:   284 | 293 | 459
//   fp32, head dim 64:   1 x 96 x 64, 13:    265 | 173 | 131    1 x 448 x 64, 13:  407 | 270 | 313
//                        4 x 448 x 64, 13:   915 | 824 | 1,076
//   fp32, head dim 128:  1 x 448 x 64, 13:   765 | 539 | -      4 x 448 x 64, 13: 1,788 | 1,770 | -
// (four groups of fp32 at head dim 128 do not fit LDS).  Lists of nearly equal length, of the
// local branch, n = 0 or half of the blocks selected and more, have hardly a popular block to wait
// for and pay only while SIMDs are idle: 4 x 24 x 128, all 24 attended, fp32, head dim 64 unsplit
// 598, pairs 560; 16 x 24 x 128 1,060 and 1,099.  With three quarters attended and more the bound
// of fp32 is lower still: head dim 64, 8 x 18 x 100, all attended, 1,152 row wavefronts in pairs, 438
// and 376, 16 x 15 x 100, 13 attended, 1,920 of them, 342 and 354 (8 attended 275 and 244); head dim
// 32, 16 x 12 x 128, 9 attended, 1,536, 1.17 times as fast in pairs, 16 x 15 x 100, 13 attended, 191
// and 206; head dim 128, where a workgroup takes the LDS of a CU, blocks of one wavefront: 8 x 32
// x 16, 256, 165 and 97, 12 x 28 x 16, 336, 152 and 165 (12 x 24 x 16, 48 heads, 17 attended, 365
// and 330).
// 1,750 launches of 24 to 14,000 row wavefronts, smooth fields, noise, n = 0 and all blocks: 1.09
// to 1.28 times as fast on average by type and head dim.  Of 600 others, up to 9,000, five were
// slower than unsplit by 2 to 11 %; what the rule leaves out gains up to twice in single cases, 4 to
// 10 % on average.  The terms a + w / c are straight lines between the launches that gain and
// those that lose: few wavefronts gain from short lists already, a full chip from long ones only.
struct BwdSplit {
    int max_waves, groups;
};
template <typename T, int D>
static BwdSplit dkdv_split(const Geom& g, int64_t BKV)
{
    // most row wavefronts that four groups and two groups speed up
    constexpr bool F32 = sizeof(T) == 4, WIDE = !F32 && D == 128;
    constexpr int64_t FOUR = WIDE ? 512 : !F32 ? 2048 : D < 128 ? 1408 : 0;
    constexpr int64_t TWO = WIDE ? 1024 : !F32 ? 4096 : D < 128 ? 8192 : 2048;
    // two groups, lists of equal length (fp32, head dim 128: a workgroup to each CU)
    constexpr int64_t EQUAL_TWO = !F32 ? TWO / 4 : D == 32 ? 1700 : 1200;
    const RowSplit single(g.block_tokens, 1, WaveTile<T>::ROWS);
    const RowSplit pairs(g.block_tokens, 2, WaveTile<T>::ROWS);
    const int64_t blocks = BKV * g.n_blocks, attended = g.n_select + 1 - g.list_only;
    const int64_t one = blocks * single.chunks, two = blocks * pairs.chunks * pairs.waves;
    const int64_t pieces = g.kv_group * attended * g.block_tokens / 32;
    const bool even = g.add_dk || attended == 1 || 2 * attended > g.n_blocks;
    const bool equal = g.add_dk || attended == 1 || 4 * attended > 3 * g.n_blocks;
    const int64_t equal_two = F32 && D == 128 ? 256 * pairs.waves : EQUAL_TWO;
    if (one <= (even ? FOUR / 3 : FOUR) && pieces >= (WIDE ? 12 + one / 64 : 6 + one / 128))
        return {1, 4};
    if (two <= (equal ? equal_two : even ? TWO / 4 : TWO) &&
        pieces >= (WIDE ? 8 + two / 128 : 6 + two / 512))
        return {2, 2};
    return {BwdLimits<T, D>::MAX_WAVES, 1};
}
// dQ: its lists are all as long, so that it is split only while wavefronts have a SIMD to
// themselves.  Whole backward, us, dQ unsplit | in two groups of pairs | in four groups
// (blocks x tokens, attended blocks; one slice, white noise):
//   bf16, head dim 32:  476 x 30, 13: 30.1 | 29.0 | 27.7      864 x 30, 13:  48.5 | 46.5 | 46.5
//   bf16, head dim 64:  120 x 100, 13: 71.2 | 62.0 | 60.7     240 x 100, 17: 123 | 118 | 127
//   bf16, head dim 128: 476 x 30, 13: 66.4 | 61.4 | -         1,000 x 30, 17: 137 | 120 | -
//   fp32, head dim 32:  120 x 64, 13: 67.5 | 56.7 | 57.3      240 x 64, 17:  115 | 113 | 120
//   fp32, head dim 64:  120 x 64, 13: 122 | 104 | 113         240 x 64, 17:  217 | 214 | 249
// Blocks of one fp32 wavefront, up to 16 tokens, form no pairs, and rounds of 64 keys are too
// long for few keys once CUs have to take several workgroups (head dim 128: their LDS holds one):
// 864 blocks of 16, head dim 32, 13 attended 62.2 | 76.4, 15 attended 7 % faster in two groups;
// head dim 128, 480 blocks, 13 attended 124 | 133, 280, 15 attended 112 | 119, 17 attended as fast,
// 240, 13 attended 86 | 78.
template <typename T, int D>
static BwdSplit dq_split(const Geom& g, int64_t BH)
{
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int64_t FOUR = D == 128 ? 0 : F32 && D == 64 ? 256 : 512;
    constexpr int64_t TWO = F32 && D == 128 ? 512 : 1024;
    const RowSplit single(g.block_tokens, 1, WaveTile<T>::ROWS);
    const int64_t waves = BH * g.n_blocks * single.chunks;
    const int64_t pieces = (g.n_select + 1 - g.list_only) * (int64_t)g.block_tokens / 32;
    if (waves <= FOUR && pieces >= 6) return {1, 4};
    const bool lone = F32 && single.chunks == 1;
    const int least = lone && D == 128 && waves > 256 ? 8 : lone && D == 32 && waves > 512 ? 7 : 5;
    return waves <= TWO && pieces >= least ? BwdSplit{2, 2} : BwdSplit{BwdLimits<T, D>::MAX_WAVES, 1};
}
template <typename T, int D, int SPLIT, bool MIXED = false>
static auto dkdv_kernel(int waves)
{
    if constexpr (SPLIT == 4) {                       // (fp32, head dim 128: not chosen)
        return bwd_generic_dkdv<T, D, 1, sizeof(T) == 4 && D == 128 ? 2 : 4>;
    } else if constexpr (SPLIT == 2) {
        return waves >= 2 ? bwd_generic_dkdv<T, D, 2, 2> : bwd_generic_dkdv<T, D, 1, 2>;
    } else {
        return waves >= 4 ? bwd_generic_dkdv<T, D, 4, 1, MIXED>
               : waves >= 2 ? bwd_generic_dkdv<T, D, 2, 1, MIXED>
                            : bwd_generic_dkdv<T, D, 1, 1, MIXED>;
    }
}
template <typename T, int D, int SPLIT, bool MIXED = false>
static auto dq_kernel(int waves)
{
    if constexpr (SPLIT == 4) {                       // (head dim 128: not chosen)
        return bwd_generic_dq<T, D, 1, D == 128 ? 2 : 4>;
    } else if constexpr (SPLIT == 2) {
        return waves >= 2 ? bwd_generic_dq<T, D, 2, 2> : bwd_generic_dq<T, D, 1, 2>;
    } else {
        // three wavefronts at head dim 128: two workgroups fit a CU, and 256 registers let
        // their six wavefronts share its SIMDs (dQ of 8 x 10 tiles -25 %; 2 x 2 wavefronts have
        // a SIMD each and take as many as they want)
        return waves >= 4 ? bwd_generic_dq<T, D, 4, 1, MIXED>
               : waves == 3 && D == 128 ? bwd_generic_dq<T, D, D == 128 ? 3 : 2, 1, MIXED>
               : waves >= 2 ? bwd_generic_dq<T, D, 2, 1, MIXED>
                            : bwd_generic_dq<T, D, 1, 1, MIXED>;
    }
}

template <typename T, int D>
static hipError_t launch_bwd_t(const void* q, const void* k, const void* v, const void* out,
                               const float* lse, const void* dout, const int32_t* sel_idx, void* dq,
                               void* dk, void* dv, float* delta, float* lse2, uint32_t* conn,
                               int32_t* order, const Geom& g, int64_t BH, hipStream_t stream)
{
    const int m = g.n_blocks, words = (m + 31) >> 5;
    const int64_t BKV = BH / g.kv_group, N = g.n_tokens;
    const bool dkdv_first = order != nullptr;        // `order` may lie where dQ goes
    const BwdSplit split_kv = dkdv_split<T, D>(g, BKV);
    const RowSplit rows_kv(g.block_tokens, split_kv.max_waves, WaveTile<T>::ROWS);
    const int waves_kv = rows_kv.waves * split_kv.groups;
    const int64_t wgs_kv = (int64_t)m * rows_kv.chunks;           // per slice
    const size_t lds_kv = sizeof(uint32_t) * (size_t)g.block_tokens;
    auto kernel_kv = split_kv.groups == 4   ? dkdv_kernel<T, D, 4>(rows_kv.waves)
                     : split_kv.groups == 2 ? dkdv_kernel<T, D, 2>(rows_kv.waves)
                     : rows_kv.narrow       ? dkdv_kernel<T, D, 1, sizeof(T) == 2>(rows_kv.waves)
                                            : dkdv_kernel<T, D, 1>(rows_kv.waves);
    const bool even = even_lists(g);
    if (even || (order && needs_no_order(kernel_kv, BKV * wgs_kv, waves_kv, lds_kv,
                                         short_lists(g, D, sizeof(T) == 4)))) order = nullptr;
    hipError_t e = launch_bwd_prepare(sizeof(T) == 2, out, dout, lse, delta, lse2, sel_idx, conn,
                                      order, g, D, BH, stream);
    if (e != hipSuccess) return e;
    auto run_dkdv = [&] {
        return launch_slices(BKV, wgs_kv * 64 * waves_kv, [&](int64_t first, int64_t slices) {
            const int64_t bh = first * g.kv_group, row = bh * N, kv = first * N * D;
            Geom piece = g;
            piece.deal = key_deal(g.deal, 2 * N * D * (int)sizeof(T), order != nullptr, even);
            if (g.add_dk) piece.add_dk += first * m * D;
            if (g.add_dv) piece.add_dv += first * m * D;
            kernel_kv<<<dim3((unsigned)(slices * wgs_kv)), dim3(64 * waves_kv), lds_kv, stream>>>(
                (const T*)q + row * D, (const T*)k + kv, (const T*)v + kv, (const T*)dout + row * D,
                lse2 + row, delta + row, conn + bh * words * m, order ? order + first * m : nullptr,
                (T*)dk + kv, (T*)dv + kv, piece, (uint32_t)slices, rows_kv.chunks,
                WaveTile<T>::ROWS * rows_kv.waves);
            return hipGetLastError();
        });
    };
    auto run_dq = [&] {
        const BwdSplit split = dq_split<T, D>(g, BH);
        const RowSplit rows(g.block_tokens, split.max_waves, WaveTile<T>::ROWS);
        const int64_t wgs = (int64_t)m * rows.chunks;
        const int nw = rows.waves * split.groups;
        auto kernel = split.groups == 4 ? dq_kernel<T, D, 4>(rows.waves)
                      : split.groups == 2 ? dq_kernel<T, D, 2>(rows.waves)
                      : rows.narrow       ? dq_kernel<T, D, 1, sizeof(T) == 2>(rows.waves)
                                          : dq_kernel<T, D, 1>(rows.waves);
        const dim3 block(64 * nw);
        return launch_slices(BKV, g.kv_group * wgs * 64 * nw, [&](int64_t first, int64_t slices) {
            const int64_t bh = first * g.kv_group, row = bh * N, kv = first * N * D;
            Geom piece = g;
            if (g.add_dq) piece.add_dq += bh * m * D;
            kernel<<<dim3((unsigned)(slices * g.kv_group * wgs)), block,
                     flat_table_bytes(g, g.n_select + 1, 1, split.groups > 2 ? 128 : 64), stream>>>(
                (const T*)q + row * D, (const T*)k + kv, (const T*)v + kv, (const T*)dout + row * D,
                lse2 + row, delta + row, sel_idx + bh * m * g.n_select, (T*)dq + row * D, piece,
                (uint32_t)slices, rows.chunks, WaveTile<T>::ROWS * rows.waves);
            return hipGetLastError();
        });
    };
    // without the memory for an order dK and dV may lie where k and v are
    e = dkdv_first ? run_dkdv() : run_dq();
    if (e != hipSuccess) return e;
    return dkdv_first ? run_dq() : run_dkdv();
}

hipError_t launch_bwd(bool is_bf16, const void* q, const void* k, const void* v, const void* out,
                      const float* lse, const void* dout, const int32_t* sel_idx, void* dq,
                      void* dk, void* dv, float* delta, float* lse2, uint32_t* conn, int32_t* order,
                      const Geom& g, int D, int64_t BH, hipStream_t stream)
{
#define BSA_CASE(DD)                                                                             \
    case DD:                                                                                     \
        return is_bf16 ? launch_bwd_t<uint16_t, DD>(q, k, v, out, lse, dout, sel_idx, dq, dk,    \
                                                    dv, delta, lse2, conn, order, g, BH, stream) \
                       : launch_bwd_t<float, DD>(q, k, v, out, lse, dout, sel_idx, dq, dk, dv,   \
                                                 delta, lse2, conn, order, g, BH, stream);
    switch (D) {
        BSA_CASE(32)
        BSA_CASE(64)
        BSA_CASE(128)
    }
#undef BSA_CASE
    return hipErrorInvalidValue;
}

}  // namespace bsa
