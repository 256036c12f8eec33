// Block selection for block-sparse attention on gfx950:
//   pool_kernel    mean-pooled block representations of Q and K (pooling
//                  equation, phi = mean);
//   select_block   block-level scores (block-level attention equation, in its
//                  rank-equivalent raw dot-product form) and the top-n key
//                  blocks of every query block (Selection paragraph);
//   pool_select_kernel  both in one launch: the pooling of one part of the
//                  batch beside the ranking of the part pooled just before.
// The scores of a query block live in LDS between the two phases of
// select_block and nowhere else: nothing of the m x m score matrix reaches HBM.
//
// The arithmetic is pinned so that the emitted indices are reproducible bit
// for bit by a scalar loop: pooled sums are fp32 adds in in-tile row-major
// order followed by one multiply by 1/b; a score is the fp32 chain
// acc = fma(qbar[d], kbar[d], acc) for d ascending from +0; candidates are
// ranked by (score descending, block index ascending) and the query block
// itself is never a candidate.  Of the matrix instructions only those of one product
// per element (fp32, K = 1) keep that chain: bsa_rank.h, for many blocks; the others
// sum in an order that cannot be reproduced by such a loop.
#include "bsa_coarse.h"
#include "bsa_device.h"
#include "bsa_launch.h"
#include "bsa_rank.h"

namespace bsa {

// ---------------------------------------------------------------------------
// pooling
// ---------------------------------------------------------------------------
// A work item is (tile, group of VEC channels); it walks the tile's tokens in
// in-tile row-major order, which is the pinned summation order.  The items of
// one (tensor, batch*head) are numbered tile-major and dealt to workgroups of
// 256 in order: consecutive lanes take consecutive channel groups, so every
// load covers whole 128-byte lines and the tiles of a tile row (bw*D elements
// each, contiguous in memory) are consumed side by side.
// `vblock` numbers the workgroups of one pooling pass: (slice, chunk of 256
// items), the n_q query slices from q_first on, then the n_k key slices from
// k_first on (fewer under grouped query attention).
template <typename T, int VEC>
__device__ __forceinline__ void pool_block(const T* __restrict__ q, const T* __restrict__ k,
                                           float* __restrict__ qbar, float* __restrict__ kbar,
                                           float* __restrict__ kbar_il,
                                           const Geom& g, int D, int64_t q_first, int64_t n_q,
                                           int64_t k_first, int wgs_per_slice, uint32_t vblock)
{
    const int chunk = (int)(vblock % (uint32_t)wgs_per_slice);
    int64_t bh_idx = vblock / (uint32_t)wgs_per_slice;
    const bool is_k = bh_idx >= n_q;
    bh_idx = is_k ? bh_idx - n_q + k_first : bh_idx + q_first;
    const T* __restrict__ x = is_k ? k : q;
    float* __restrict__ xbar = is_k ? kbar : qbar;
    const int groups = D / VEC;
    const int items = g.n_blocks * groups;
    const float inv_b = 1.0f / (float)g.block_tokens;
    x += bh_idx * g.n_tokens * D;

    const int item = chunk * 256 + (int)threadIdx.x;
    if (item >= items) return;
    const int beta = item / groups;
    const int ch = (item - beta * groups) * VEC;
    const int tile_row = beta / g.blocks_per_row, tile_col = beta - tile_row * g.blocks_per_row;
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.0f;
    for (int rr = 0; rr < g.block_h; ++rr) {
        const T* row = x + ((int64_t)(tile_row * g.block_h + rr) * g.grid_w +
                            (int64_t)tile_col * g.block_w) * D + ch;
#pragma unroll 8
        for (int cc = 0; cc < g.block_w; ++cc) {
#pragma unroll
            for (int e4 = 0; e4 < VEC; e4 += 4) {
                // streamed: every byte is used once here, nothing is worth caching
                const float4 v = load4_stream(row + (int64_t)cc * D + e4);
                acc[e4 + 0] = acc[e4 + 0] + v.x;
                acc[e4 + 1] = acc[e4 + 1] + v.y;
                acc[e4 + 2] = acc[e4 + 2] + v.z;
                acc[e4 + 3] = acc[e4 + 3] + v.w;
            }
        }
    }
    float* dst = xbar + (bh_idx * g.n_blocks + beta) * D + ch;
#pragma unroll
    for (int e4 = 0; e4 < VEC; e4 += 4)
        store4(dst + e4, make_float4(acc[e4] * inv_b, acc[e4 + 1] * inv_b,
                                     acc[e4 + 2] * inv_b, acc[e4 + 3] * inv_b));
    // second copy of the pooled keys for the ranking, per slice [D/4][m][4]: a
    // wavefront whose lanes hold 64 consecutive key blocks then reads 1 KiB runs
    if (is_k && kbar_il) {
        float* il = kbar_il + bh_idx * g.n_blocks * D;
#pragma unroll
        for (int e4 = 0; e4 < VEC; e4 += 4)
            store4(il + ((int64_t)((ch + e4) >> 2) * g.n_blocks + beta) * 4,
                   make_float4(acc[e4] * inv_b, acc[e4 + 1] * inv_b, acc[e4 + 2] * inv_b,
                               acc[e4 + 3] * inv_b));
    }
}

// Pooling as a launch of its own (little to pool, or nothing to rank beside it):
// the same sums with more loads in flight.  A thread owns VEC channels of a tile and
// walks the tile's tokens BATCH at a time, over row ends, all loads of a batch
// before the adds.  VEC is chosen by the launcher: 16 bytes per load where that
// fills the chip, less where it would leave too few wavefronts: what bounds a
// small call is the number of memory latencies in a thread's chain.
// Measured against pool_block in a launch of its own (16-byte loads, 8 in flight):
// 25 slices of 24 tiles of 128 tokens (10 MB) 12.1 -> 6.5 us; 32 slices of 288 tiles
// of 10 x 10 (118 MB) 24.3 -> 23.3 us, which is the memory's rate, as is 10.8 us for
// 59 MB.
template <typename T, int VEC> struct PoolPiece { T x[VEC]; };

template <int VEC>
__device__ __forceinline__ void add_piece(const PoolPiece<uint16_t, VEC>& p, float (&acc)[VEC])
{
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = acc[e] + bf16_to_f32(p.x[e]);
}
template <int VEC>
__device__ __forceinline__ void add_piece(const PoolPiece<float, VEC>& p, float (&acc)[VEC])
{
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = acc[e] + p.x[e];
}

// A tensor of `slices` slices and where its means go (il: second copy of the means,
// per slice [D/4][m][4], or null).
struct PoolTensor {
    const void* x;
    float *xbar, *xbar_il;
    uint32_t slices;
};

// Block lists of the local branch: lists[bh, i, c], c = 0 .. local_h*local_w - 2, the
// other tiles of the aligned group of local_h x local_w tiles that contains tile i,
// ascending.  Written by the workgroups of a pooling launch from first_wg on.
struct LocalLists {
    int32_t* lists;
    int32_t local_h, local_w;
    int64_t total;          // entries
    uint32_t first_wg;
};

__device__ __forceinline__ void write_local_list(const LocalLists& ll, const Geom& g)
{
    const int64_t e = (int64_t)(blockIdx.x - ll.first_wg) * 256 + threadIdx.x;
    if (e >= ll.total) return;
    const int nl = ll.local_h * ll.local_w - 1;
    const int c = (int)(e % nl);
    const int i = (int)((e / nl) % g.n_blocks);
    const int r = i / g.blocks_per_row, col = i - r * g.blocks_per_row;
    const int r0 = r - r % ll.local_h, c0 = col - col % ll.local_w;
    const int own = (r - r0) * ll.local_w + (col - c0);    // position of tile i in its group
    const int pos = c < own ? c : c + 1;
    ll.lists[e] = (r0 + pos / ll.local_w) * g.blocks_per_row + c0 + pos % ll.local_w;
}

template <typename T, int VEC>
__global__ __launch_bounds__(256) void pool_kernel(PoolTensor t0, PoolTensor t1, PoolTensor t2,
                                                   Geom g, int D, uint32_t wgs_per_slice,
                                                   LocalLists ll)
{
    typedef uint32_t word __attribute__((ext_vector_type(VEC * (int)sizeof(T) / 4)));
    constexpr int BATCH = 16;
    if (blockIdx.x >= ll.first_wg) {
        write_local_list(ll, g);
        return;
    }
    uint32_t slice = blockIdx.x / wgs_per_slice;
    const uint32_t chunk = blockIdx.x - slice * wgs_per_slice;
    PoolTensor t = t0;
    if (slice >= t.slices) {
        slice -= t.slices;
        t = t1;
        if (slice >= t.slices) { slice -= t.slices; t = t2; }
    }
    const int groups = D / VEC;
    const int item = (int)(chunk * 256 + threadIdx.x);
    const int beta = item / groups;
    if (beta >= g.n_blocks) return;
    const int ch = (item - beta * groups) * VEC;
    const int tile_row = beta / g.blocks_per_row, tile_col = beta - tile_row * g.blocks_per_row;
    const T* at = (const T*)t.x + (int64_t)slice * g.n_tokens * D +
                  ((int64_t)tile_row * g.block_h * g.grid_w + (int64_t)tile_col * g.block_w) * D + ch;
    const int64_t row_jump = (int64_t)(g.grid_w - g.block_w) * D;
    const int b = g.block_tokens;
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.0f;
    int col = 0;                                     // wave-uniform: position in the tile row
    auto next = [&] {
        const T* here = at;
        at += D;
        if (++col == g.block_w) { col = 0; at += row_jump; }
        return here;
    };
    int tau = 0;
    for (; tau + BATCH <= b; tau += BATCH) {
        word w[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const word* src = (const word*)next();
            // 16-byte pieces: much to read, once
            w[u] = sizeof(word) == 16 ? __builtin_nontemporal_load(src) : *src;
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) add_piece(__builtin_bit_cast(PoolPiece<T, VEC>, w[u]), acc);
    }
    for (; tau < b; ++tau)
        add_piece(__builtin_bit_cast(PoolPiece<T, VEC>, *(const word*)next()), acc);
    const float inv_b = 1.0f / (float)b;
    float* dst = t.xbar + ((int64_t)slice * g.n_blocks + beta) * D + ch;
    float* il = t.xbar_il ? t.xbar_il + (int64_t)slice * g.n_blocks * D : nullptr;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const float mean = acc[e] * inv_b;
        dst[e] = mean;
        if (il) il[((int64_t)((ch + e) >> 2) * g.n_blocks + beta) * 4 + ((ch + e) & 3)] = mean;
    }
}

// ---------------------------------------------------------------------------
// scores + top-n
// ---------------------------------------------------------------------------
// Top-n of one row of m ranking keys (in LDS) by one wavefront; cand: 64 words of LDS
// of its own.  A round finds a threshold that at least `want` lanes' best keys reach
// (bit by bit, 20 of the 32 bits: a lower threshold only lets more through), collects
// the candidates at or above it, which are therefore the best `count` >= want of all,
// as composites (key << 32 | ~j) that are distinct and order exactly as the ranking
// does, and places each by counting the larger ones.  On smooth scores a round of
// 16 collects about 20 candidates.  Rounds repeat until n are placed.
// Clustered scores (equal in their upper 20 bits) show in the number of lanes that
// reach the threshold, which then gets all 32 bits.  Equal scores: if the threshold
// is the largest key itself, its blocks are placed as they come, in ascending order;
// if more than 64 candidates reach it, those above it are taken.  Otherwise more than
// 64 mean that half as many are wanted (32 at first, 16 for most rows).
// Ranking and pooling, n = 32: equal scores 450 blocks x 8 heads 120 -> 30 us, 4,096
// x 4 3,770 -> 177; clustered 120 -> 33 and 3,810 -> 346; smooth 33.3 -> 33.5 and
// 340 -> 345 (with one pick per round for equal and clustered scores before).
// About 12 vector instructions per pick against 22 with a sorted list of 8 per lane
// (m <= 512) and 110 with 64 candidates per lane (m <= 4096), and no registers that
// grow with m: ranking 8,192 rows of 1,024 (head dim 32) 57 -> 30 us, 43,200
// rows of 450, n = 16, 105 -> 84 us.
__device__ __forceinline__ void topn_of_row(uint32_t* keys, uint64_t* cand,
                                            int32_t* __restrict__ dst, int m, int n, int lane)
{
    int done = 0, limit = 32;
    // candidates with keys >= floor_key into cand (the first 64 of them); their number
    auto collect = [&](uint32_t floor_key) {
        int count = 0;
        for (int j0 = 0; j0 < m; j0 += 64) {
            const int j = j0 + lane;
            const uint32_t key = j < m ? keys[j] : 0u;
            const bool in = key >= floor_key;
            const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
            if (mask) {
                const int at = count + place_in(mask);
                if (in && at < 64) cand[at] = ((uint64_t)key << 32) | (uint32_t)~j;
                count += __builtin_popcountll(mask);
            }
        }
        return count;
    };
    while (done < n) {
        uint32_t best = 0;
        for (int j = lane; j < m; j += 64) best = max(best, keys[j]);
        const int want = min(n - done, limit);
        uint32_t floor_key = 0;
        int bit = 31;
        auto refine = [&](int last) {
            for (; bit >= last; --bit) {
                const uint32_t t = floor_key | (1u << bit);
                if (__builtin_popcountll(__builtin_amdgcn_ballot_w64(best >= t)) >= want)
                    floor_key = t;
            }
        };
        refine(12);
        if (__builtin_popcountll(__builtin_amdgcn_ballot_w64(best >= floor_key)) >= want + 8)
            refine(0);
        auto none_above = [&] { return __builtin_amdgcn_ballot_w64(best > floor_key) == 0; };
        int count = 65;
        if (bit >= 0 || !none_above()) count = collect(max(floor_key, 1u));   // 0: removed
        if (count > 64) {
            if (want == 1) refine(0);
            if (bit < 0) {
                if (none_above()) {
                    // floor_key is the largest key left
                    for (int j0 = 0; j0 < m && done < n; j0 += 64) {
                        const int j = j0 + lane;
                        const bool in = j < m && keys[j] == floor_key;
                        const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
                        if (in) {
                            const int at = done + place_in(mask);
                            if (at < n) dst[at] = j;
                            keys[j] = 0u;
                        }
                        done += __builtin_popcountll(mask);
                    }
                    continue;
                }
                count = collect(floor_key + 1);
            }
            if (count > 64) {
                limit = want >> 1;
                continue;
            }
        }
        const uint64_t mine = lane < count ? cand[lane] : 0ull;
        int rank = 0;
        for (int t = 0; t < count; ++t) {
            const uint64_t c =
                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine >> 32), t) << 32) |
                (uint32_t)__builtin_amdgcn_readlane((int)mine, t);
            rank += c > mine ? 1 : 0;
        }
        const int placed = min(count, n - done);
        const uint32_t block = ~(uint32_t)mine;
        if (lane < count) {
            if (rank < placed) dst[done + rank] = (int32_t)block;
            keys[block] = 0u;
        }
        done += placed;
        if (limit < 16) limit *= 2;
    }
}

// One workgroup of 256 threads ranks G consecutive query blocks of one
// (batch, head).
//   phase 1: thread t owns key block j = t, t + 256, ..., holds kbar_j in
//            registers (loaded from the channel-interleaved copy of the pooled
//            keys: consecutive lanes read consecutive 16-byte groups) and runs the pinned fma chain against each of the
//            G pooled queries (wave-uniform: scalar loads, scalar operands); the
//            ranking keys of all m candidates of each query land in LDS.
//   phase 2: one wavefront per query block, topn_of_row.
// LDS: G*m u32 (ranking keys) and the candidates of four rows.  BIG: the variant for
// m > 512, which gives a thread two key blocks at a time (a kernel of its own: its
// register count must not cost the common case its occupancy).
template <int D, bool BIG>
__device__ __forceinline__ void select_block(const float* __restrict__ qbar,
                                             const float* __restrict__ kbar_il,
                                             int32_t* __restrict__ sel_idx, const Geom& g, int G,
                                             uint32_t vblock)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint32_t* key_s = (uint32_t*)smem;               // [G][m]
    __shared__ uint64_t cand_s[4][64];

    const int m = g.n_blocks, n = g.n_select;
    // vblock = batch*head * groups + group
    const int groups = (m + G - 1) / G;
    const int64_t bh_idx = vblock / (uint32_t)groups;
    const int i0 = (int)(vblock - (uint32_t)bh_idx * (uint32_t)groups) * G;
    const int rows = min(G, m - i0);
    qbar += (bh_idx * m + i0) * D;
    kbar_il += kv_slice_of(g, bh_idx) * m * D;       // per slice [D/4][m][4]

    // ---- phase 1: scores.  The pooled queries are wave-uniform and are fetched
    // with scalar loads straight into the fma's scalar operand.
    auto load_key = [&](int j, float (&kr)[D]) {
        const float4* ksrc = (const float4*)kbar_il + j;
#pragma unroll
        for (int d4 = 0; d4 < D / 4; ++d4) {
            const float4 v = ksrc[(int64_t)d4 * m];
            kr[4 * d4 + 0] = v.x; kr[4 * d4 + 1] = v.y;
            kr[4 * d4 + 2] = v.z; kr[4 * d4 + 3] = v.w;
        }
    };
    auto put_key = [&](int r, int j, float acc) {
        key_s[r * m + j] = (j == i0 + r && !g.own_is_candidate) ? 0u : rank_key(acc);
    };
    int j = threadIdx.x;
    if constexpr (BIG && D <= 64) {
        // Two key blocks per thread at a time: with this many blocks the LDS rows
        // leave one workgroup per CU, i.e. one wavefront per SIMD, and the two
        // independent chains (same scalar operand) hide the latency of one.
        for (; j + (int)blockDim.x < m; j += 2 * (int)blockDim.x) {
            float ka[D], kb[D];
            load_key(j, ka);
            load_key(j + (int)blockDim.x, kb);
            for (int r = 0; r < rows; ++r) {
                const float* __restrict__ qrow = qbar + r * D;
                float a = 0.0f, b = 0.0f;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    a = __builtin_fmaf(qrow[d], ka[d], a);
                    b = __builtin_fmaf(qrow[d], kb[d], b);
                }
                put_key(r, j, a);
                put_key(r, j + (int)blockDim.x, b);
            }
        }
    }
    for (; j < m; j += blockDim.x) {
        float kr[D];
        load_key(j, kr);
        for (int r = 0; r < rows; ++r) {
            const float* __restrict__ qrow = qbar + r * D;
            float acc = 0.0f;
#pragma unroll
            for (int d = 0; d < D; ++d) acc = __builtin_fmaf(qrow[d], kr[d], acc);
            put_key(r, j, acc);
        }
    }
    __syncthreads();

    // ---- phase 2: top-n per query block, one wavefront each
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int r = wave; r < rows; r += (int)(blockDim.x >> 6))
        topn_of_row(key_s + r * m, cand_s[wave], sel_idx + ((bh_idx * m) + i0 + r) * n, m, n, lane);
}

// Pooling of one part of the batch beside the ranking of the part pooled by
// the launch before: pooling is bound by HBM and leaves the vector ALUs idle,
// the ranking is bound by the vector ALUs and reads only cached pooled means.
// The first n_poolers workgroups of the launch pool: they are dispatched
// first and each walks the part's n_pool_blocks pooling blocks with stride
// n_poolers, so a fixed number of them stays resident on every CU until the
// part is pooled (pooling workgroups dealt one block each are short-lived and
// would be crowded out by the long-lived ranking workgroups).  The other
// workgroups rank (virtual ids from select_first on).  No workgroup waits for
// another: what a ranking workgroup reads was written by an earlier launch.
// The pooled means are passed twice: written through qbar_w / kbar_w / kbar_il_w
// (the part being pooled), read through qbar_r / kbar_il_r (the part
// being ranked).
template <typename T, int VEC, int D, int MODE>
__global__ __launch_bounds__(256, MODE == 2 ? 2 : 1) void pool_select_kernel(
    const T* __restrict__ q, const T* __restrict__ k, float* __restrict__ qbar_w,
    float* __restrict__ kbar_w, float* __restrict__ kbar_il_w, const float* __restrict__ qbar_r,
    const float* __restrict__ kbar_il_r,
    int32_t* __restrict__ sel_idx, Geom g, int G,
    int64_t pool_q_first, int64_t pool_n_q, int64_t pool_k_first, int wgs_per_slice,
    uint32_t n_pool_blocks, uint32_t n_poolers, uint32_t select_first)
{
    if (blockIdx.x >= n_poolers) {
        const uint32_t vblock = select_first + (blockIdx.x - n_poolers);
        if constexpr (MODE == 2) {
            extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
            rank_block<D>(qbar_r, kbar_il_r, sel_idx, g, G, vblock, *(RankShared<D>*)smem);
        } else {
            select_block<D, MODE == 1>(qbar_r, kbar_il_r, sel_idx, g, G, vblock);
        }
        return;
    }
    for (uint32_t v = blockIdx.x; v < n_pool_blocks; v += n_poolers)
        pool_block<T, VEC>(q, k, qbar_w, kbar_w, kbar_il_w, g, D, pool_q_first, pool_n_q, pool_k_first,
                           wgs_per_slice, v);
}

// The ranking beside the coarse branch, for a batch that is pooled by a launch of its
// own: both read only pooled means, and apart each would leave most of the chip idle
// (of a small batch).  Workgroups below n_rank rank.
template <int D, int MODE>
__global__ __launch_bounds__(256) void rank_coarse_kernel(
    const float* __restrict__ qbar, const float* __restrict__ kbar_il,
    const float* __restrict__ vbar, float* __restrict__ obar, int32_t* __restrict__ sel_idx, Geom g,
    int G, int G_coarse, uint32_t n_rank)
{
    if (blockIdx.x < n_rank)
        select_block<D, MODE == 1>(qbar, kbar_il, sel_idx, g, G, blockIdx.x);
    else
        coarse_block<D>(qbar, kbar_il, vbar, obar, g, G_coarse, blockIdx.x - n_rank);
}

// ---------------------------------------------------------------------------
// Checker for caller-made selections (the attention kernels trust sel_idx):
// one thread per row counts the entries that are out of range, repeat an
// earlier entry of the row or, unless own_ok, name the row's own block.
// ---------------------------------------------------------------------------
__global__ void zero_counter_kernel(int32_t* counter) { *counter = 0; }

__global__ __launch_bounds__(256) void check_selection_kernel(const int32_t* __restrict__ sel_idx,
                                                              int32_t* __restrict__ n_bad, Geom g,
                                                              int own_ok, int64_t rows)
{
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int bad = 0;
    if (row < rows) {
        const int n = g.n_select, m = g.n_blocks;
        const int own = (int)(row % m);
        const int32_t* r = sel_idx + row * n;
        for (int a = 0; a < n; ++a) {
            const int32_t x = r[a];
            bool is_bad = x < 0 || x >= m || (!own_ok && x == own);
            for (int c = 0; c < a && !is_bad; ++c) is_bad = r[c] == x;
            bad += is_bad ? 1 : 0;
        }
    }
    // one integer atomic per wavefront with something to report
    for (int off = 32; off >= 1; off >>= 1) bad += __shfl_xor(bad, off);
    if ((threadIdx.x & 63) == 0 && bad) atomicAdd(n_bad, bad);
}

hipError_t launch_check_selection(const int32_t* sel_idx, int32_t* n_bad, const Geom& g,
                                  bool own_ok, int64_t BH, hipStream_t stream)
{
    hipLaunchKernelGGL(zero_counter_kernel, dim3(1), dim3(1), 0, stream, n_bad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || g.n_select == 0) return e;
    const int64_t rows = BH * g.n_blocks;
    hipLaunchKernelGGL(check_selection_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0,
                       stream, sel_idx, n_bad, g, own_ok ? 1 : 0, rows);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
static constexpr size_t kSelectLdsBudget = 144 * 1024;

static size_t select_lds_bytes(int G, int m)
{
    return (size_t)G * (size_t)m * 4;
}

int select_group_size(int m)
{
    // the largest G in [1, 8] whose LDS footprint fits, and fits twice where
    // that is possible with G >= 4 (two workgroups per CU cover each other's
    // loads, and a pooling workgroup fits beside a ranking one); 0 if even
    // G = 1 does not fit
    for (int G = 8; G >= 4; G >>= 1)
        if (2 * select_lds_bytes(G, m) <= kSelectLdsBudget) return G;
    for (int G = 8; G >= 1; G >>= 1)
        if (select_lds_bytes(G, m) <= kSelectLdsBudget) return G;
    return 0;
}

template <typename T, int VEC>
static hipError_t launch_pool_t(const PoolTensor (&t)[3], LocalLists ll, const Geom& g, int D,
                                hipStream_t stream)
{
    const int64_t slices = (int64_t)t[0].slices + t[1].slices + t[2].slices;
    const int64_t wgs_per_slice = ((int64_t)g.n_blocks * (D / VEC) + 255) / 256;
    const int64_t wgs = slices * wgs_per_slice, list_wgs = (ll.total + 255) / 256;
    if (wgs + list_wgs >= (int64_t)1 << 31) return hipErrorInvalidValue;
    ll.first_wg = (uint32_t)wgs;
    pool_kernel<T, VEC><<<dim3((unsigned)(wgs + list_wgs)), dim3(256), 0, stream>>>(
        t[0], t[1], t[2], g, D, (uint32_t)wgs_per_slice, ll);
    return hipGetLastError();
}

// Pools up to three tensors.  16-byte loads when that gives every CU two
// workgroups of 256 threads, else 8 or 4 bytes.
static hipError_t launch_pool_tensors(bool is_bf16, const PoolTensor (&t)[3], const LocalLists& ll,
                                      const Geom& g, int D, hipStream_t stream)
{
    const int64_t slices = (int64_t)t[0].slices + t[1].slices + t[2].slices;
    const int64_t channels = slices * g.n_blocks * D;
    const int64_t fill = (int64_t)2 * 256 * 256;             // threads
    const int per16 = is_bf16 ? 8 : 4;
    if (channels / per16 >= fill)
        return is_bf16 ? launch_pool_t<uint16_t, 8>(t, ll, g, D, stream)
                       : launch_pool_t<float, 4>(t, ll, g, D, stream);
    if (2 * channels / per16 >= fill)
        return is_bf16 ? launch_pool_t<uint16_t, 4>(t, ll, g, D, stream)
                       : launch_pool_t<float, 2>(t, ll, g, D, stream);
    return is_bf16 ? launch_pool_t<uint16_t, 2>(t, ll, g, D, stream)
                   : launch_pool_t<float, 1>(t, ll, g, D, stream);
}

hipError_t launch_pool(bool is_bf16, const void* q, const void* k, float* qbar, float* kbar,
                       const Geom& g, int D, int64_t BH, hipStream_t stream)
{
    const PoolTensor t[3] = {{q, qbar, nullptr, (uint32_t)BH},
                             {k, kbar, nullptr, (uint32_t)(BH / g.kv_group)},
                             {nullptr, nullptr, nullptr, 0}};
    return launch_pool_tensors(is_bf16, t, LocalLists{}, g, D, stream);
}

size_t select_scratch_bytes(int m, int D, int64_t BKV)
{
    // the ranking reads a second, channel-interleaved copy of the pooled keys
    return (size_t)BKV * (size_t)m * (size_t)D * 4;
}

// pooling workgroups that stay resident beside the ranking (one per CU)
constexpr int64_t kPoolers = 256;

// Parts of the batch: as many as leave each about 128 MiB to pool, at most 4.  A
// part costs a launch that the GPU drains before the next one (8 us and more),
// and what it buys is the shorter of pooling and ranking of a part.  Measured with
// 1 / 2 / 4 parts: 59 MB (1.5 degree grid, 8 heads) 28 / 40 / 63 us, 118 MB 36 / 44
// / 67, 252 MB 79 / 73 / 84, 944 MB 237 / 229 / 203, 2.8 GB (24 members) 862 / 749
// / 705.
constexpr int64_t kPartBytes = (int64_t)128 << 20;
constexpr int64_t kMaxParts = 4;

static int select_parts(int64_t BH, int64_t BKV, const Geom& g, int D, size_t element)
{
    const int64_t bytes = (BH + BKV) * g.n_tokens * D * (int64_t)element;
    int64_t parts = (bytes + kPartBytes / 2) / kPartBytes;
    if (parts > kMaxParts) parts = kMaxParts;
    if (parts > BKV) parts = BKV;
    return parts < 1 ? 1 : (int)parts;
}

// Few query blocks: fewer per workgroup, down to a workgroup each, until there are
// two workgroups per CU (ranking 480 blocks 9.8 -> 5.1 us, 3,600 blocks 15.9 -> 13.4
// us, 64 blocks 6.3 -> 3.9 us).
static int select_group_for(int m, int64_t BH)
{
    int G = select_group_size(m);
    while (G > 1 && BH * ((m + G - 1) / G) < 512) G >>= 1;
    return G;
}

// Which code ranks: 2 rank_block, 1 select_block for many blocks, 0 select_block.
// rank_block, 32 query blocks to a workgroup, takes long for a workgroup (25 us and 5 to 10
// per 256 blocks) and pays where the pooled keys are large and the workgroups fill the
// chip.  select_block over rank_block, ranking alone, smooth fields, noise, equal scores,
// rising scores: head dim 32, 16 slices of 2,048 blocks 1.6, 1.4, 1.1, 1.2, of 1,012 0.8,
// 0.9, 0.6, 0.7; 64, 16 of 2,048 1.6, 1.5, 1.2, 1.2, of 1,012 1.1, 1.2, 0.8, 1.0, 4 of 2,048
// 1.2, 1.2, 0.9, 0.8; 128, 16 of 1,012 1.4, 1.5, 1.2, 1.3, 4 of 2,048 1.5, 1.4, 1.3, 1.2, 16
// of 512 1.0, 1.1, 0.9, 0.8 (n = 16; n = 64 on rising scores 0.6 to 0.9).
static int64_t rank_workgroups(int m, int64_t BH) { return BH * ((m + kRankRows - 1) / kRankRows); }
static int rank_mode(const Geom& g, int D, int64_t BH)
{
    const int m = g.n_blocks, n = g.n_select;
    if (n >= 1 && n <= kRankPicks && (int64_t)m * D >= 98304 && rank_workgroups(m, BH) * D >= 30000)
        return 2;
    return m > 512 ? 1 : 0;
}

// About 0.62 of the steps of rank_block, coprime to their number.
static int rank_stride(int m)
{
    const int steps = (m + 255) / 256;
    auto gcd = [](int a, int b) {
        while (b) { const int t = a % b; a = b; b = t; }
        return a;
    };
    int stride = steps * 5 / 8;
    if (stride < 1) stride = 1;
    while (gcd(stride, steps) != 1) ++stride;
    return stride;
}

template <typename T, int VEC, int D, int MODE>
static hipError_t launch_pool_select_t(const void* q, const void* k, float* qbar, float* kbar,
                                       float* kbar_il, int32_t* sel_idx, const Geom& g,
                                       int64_t BH, bool pooled, hipStream_t stream)
{
    const int m = g.n_blocks;
    // G: query blocks per workgroup, or the stride of the groups of keys (rank_block)
    const int G = MODE == 2 ? rank_stride(m) : select_group_for(m, BH);
    if (G == 0) return hipErrorInvalidValue;
    const size_t lds = MODE == 2 ? sizeof(RankShared<D>) : select_lds_bytes(G, m);
    // the attribute is per device; setting it twice (two host threads racing) is harmless
    static bool attr_set[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!attr_set[dev]) {
        hipError_t e = hipFuncSetAttribute((const void*)pool_select_kernel<T, VEC, D, MODE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kSelectLdsBudget);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    const int64_t BKV = BH / g.kv_group;
    int parts = pooled ? 1 : select_parts(BH, BKV, g, D, sizeof(T));
    // rank_block: parts that fill the chip with workgroups of several steps (24 slices of 2,276
    // blocks, head dim 128, 1 / 2 / 3 / 4 parts 769 / 774 / 887 / 964 us; 16 of 3,422, head dim
    // 64, 659 / 647 / 649 / 606)
    if (MODE == 2)
        while (parts > 1 && rank_workgroups(m, BH) < (int64_t)parts * 6 * D) --parts;
    const int wgs_per_slice = (m * (D / VEC) + 255) / 256;
    const int groups = MODE == 2 ? (m + kRankRows - 1) / kRankRows : (m + G - 1) / G;
    // one part: pooled by a launch of its own
    if (parts == 1 && !pooled) {
        const PoolTensor tensors[3] = {{q, qbar, nullptr, (uint32_t)BH},
                                       {k, kbar, kbar_il, (uint32_t)BKV},
                                       {nullptr, nullptr, nullptr, 0}};
        const hipError_t e = launch_pool_tensors(sizeof(T) == 2, tensors, LocalLists{}, g, D, stream);
        if (e != hipSuccess) return e;
    }
    // launch t pools part t and ranks part t - 1
    for (int t = parts == 1 ? 1 : 0; t <= parts; ++t) {
        int64_t pq0 = 0, pnq = 0, pk0 = 0, n_pool = 0, sel_first = 0, n_sel = 0;
        if (t < parts) {
            pk0 = BKV * t / parts;
            const int64_t pk1 = BKV * (t + 1) / parts;
            pq0 = pk0 * g.kv_group;
            pnq = (pk1 - pk0) * g.kv_group;
            n_pool = (pnq + (pk1 - pk0)) * wgs_per_slice;
        }
        if (t >= 1) {
            const int64_t k0 = BKV * (t - 1) / parts, k1 = BKV * t / parts;
            sel_first = k0 * g.kv_group * groups;
            n_sel = (k1 - k0) * g.kv_group * groups;
        }
        if (n_pool + n_sel == 0) continue;
        // alone, the pooling blocks get a workgroup each
        const int64_t n_poolers = n_sel == 0 ? n_pool : (n_pool < kPoolers ? n_pool : kPoolers);
        if (n_pool >= ((int64_t)1 << 31) || n_poolers + n_sel >= ((int64_t)1 << 31) ||
            sel_first + n_sel >= ((int64_t)1 << 32))
            return hipErrorInvalidValue;
        hipLaunchKernelGGL((pool_select_kernel<T, VEC, D, MODE>), dim3((unsigned)(n_poolers + n_sel)),
                           dim3(256), lds, stream, (const T*)q, (const T*)k, qbar, kbar, kbar_il,
                           (const float*)qbar, (const float*)kbar_il, sel_idx,
                           g, G, pq0, pnq, pk0,
                           wgs_per_slice, (uint32_t)n_pool, (uint32_t)n_poolers,
                           (uint32_t)sel_first);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_pool_select(bool is_bf16, const void* q, const void* k, float* qbar,
                              float* kbar, void* scratch, int32_t* sel_idx, const Geom& g, int D,
                              int64_t BH, bool pooled, hipStream_t stream)
{
    // the channel-interleaved copy of the pooled keys
    float* il = (float*)scratch;
    if (!il) return hipErrorInvalidValue;
    const int mode = rank_mode(g, D, BH);
#define BSA_PS(T, VEC, D_)                                                                        \
    (mode == 2   ? launch_pool_select_t<T, VEC, D_, 2>(q, k, qbar, kbar, il, sel_idx, g, BH,      \
                                                       pooled, stream)                            \
     : mode == 1 ? launch_pool_select_t<T, VEC, D_, 1>(q, k, qbar, kbar, il, sel_idx, g, BH,      \
                                                       pooled, stream)                            \
                 : launch_pool_select_t<T, VEC, D_, 0>(q, k, qbar, kbar, il, sel_idx, g, BH,      \
                                                       pooled, stream))
    switch (D) {
    case 32: return is_bf16 ? BSA_PS(uint16_t, 8, 32) : BSA_PS(float, 4, 32);
    case 64: return is_bf16 ? BSA_PS(uint16_t, 8, 64) : BSA_PS(float, 4, 64);
    case 128: return is_bf16 ? BSA_PS(uint16_t, 8, 128) : BSA_PS(float, 4, 128);
    }
#undef BSA_PS
    return hipErrorInvalidValue;
}

// The ranking shares a launch with the coarse branch unless the larger LDS rows of the
// latter would leave a ranking workgroup alone on its CU that fits twice by itself.
// Three-branch forward in one launch against two, head dim 64: 24 blocks 37 against 42
// us, 450 x 8 heads 157 / 164, 2,048 x 4 543 / 553, 8,192 x 1 2,316 / 2,379; where the
// rule parts them: 4,096 x 2 1,180 / 1,090, head dim 32 4,096 x 4 1,422 / 1,266, head
// dim 128 2,048 x 2 737 / 717.  (900 blocks at head dim 64 lose 4 % together; head dims
// 32 and 128 win 2 to 5 % there.)
static bool rank_beside_coarse(int m, int D, int64_t BH)
{
    constexpr size_t lds_of_cu = 160 * 1024, candidates = 4 * 64 * sizeof(uint64_t);
    const size_t rank = select_lds_bytes(select_group_for(m, BH), m) + candidates;
    const size_t coarse = coarse_lds_bytes(coarse_group_for(m, D, BH), m, D) + candidates;
    return 2 * coarse <= lds_of_cu || 2 * rank > lds_of_cu;
}

template <int D, int MODE>
static hipError_t launch_rank_coarse_t(const float* qbar, const float* kbar_il, const float* vbar,
                                       float* obar, int32_t* sel_idx, const Geom& g, int64_t BH,
                                       hipStream_t stream)
{
    const int m = g.n_blocks;
    const int G = select_group_for(m, BH), Gc = coarse_group_for(m, D, BH);
    if (G == 0 || Gc == 0) return hipErrorInvalidValue;
    const size_t rank_lds = select_lds_bytes(G, m), coarse_lds = coarse_lds_bytes(Gc, m, D);
    static bool attr_set[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!attr_set[dev]) {
        hipError_t e = hipFuncSetAttribute((const void*)rank_coarse_kernel<D, MODE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(kSelectLdsBudget > kCoarseLdsBudget
                                                     ? kSelectLdsBudget : kCoarseLdsBudget));
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    const int64_t n_rank = BH * ((m + G - 1) / G), n_coarse = BH * ((m + Gc - 1) / Gc);
    if (n_rank + n_coarse >= (int64_t)1 << 31) return hipErrorInvalidValue;
    rank_coarse_kernel<D, MODE><<<dim3((unsigned)(n_rank + n_coarse)), dim3(256),
                                 rank_lds > coarse_lds ? rank_lds : coarse_lds, stream>>>(
        qbar, kbar_il, vbar, obar, sel_idx, g, G, Gc, (uint32_t)n_rank);
    return hipGetLastError();
}

hipError_t launch_blocks_three_branch(bool is_bf16, const void* q, const void* k, const void* v,
                                      float* qbar, float* kbar, float* vbar, float* kbar_il,
                                      int32_t* sel_idx, float* obar, int32_t* lists, int local_h,
                                      int local_w, const Geom& g, int D, int64_t BH,
                                      hipStream_t stream)
{
    const int m = g.n_blocks;
    const int64_t BKV = BH / g.kv_group;
    const LocalLists ll = {lists, local_h, local_w, BH * m * (local_h * local_w - 1), 0};
    const PoolTensor none = {nullptr, nullptr, nullptr, 0};
    const PoolTensor tv = {v, vbar, nullptr, (uint32_t)BKV};
    if (select_parts(BH, BKV, g, D, is_bf16 ? 2 : 4) > 1) {
        hipError_t e = launch_pool_select(is_bf16, q, k, qbar, kbar, kbar_il, sel_idx, g, D, BH,
                                          false, stream);
        if (e != hipSuccess) return e;
        const PoolTensor t[3] = {tv, none, none};
        e = launch_pool_tensors(is_bf16, t, ll, g, D, stream);
        return e != hipSuccess ? e : launch_coarse(qbar, kbar_il, vbar, obar, g, D, BH, stream);
    }
    const PoolTensor t[3] = {{q, qbar, nullptr, (uint32_t)BH}, {k, kbar, kbar_il, (uint32_t)BKV}, tv};
    const hipError_t e = launch_pool_tensors(is_bf16, t, ll, g, D, stream);
    if (e != hipSuccess) return e;
    if (rank_mode(g, D, BH) == 2 || !rank_beside_coarse(m, D, BH)) {
        const hipError_t r = launch_pool_select(is_bf16, q, k, qbar, kbar, kbar_il, sel_idx, g, D, BH,
                                                true, stream);
        return r != hipSuccess ? r : launch_coarse(qbar, kbar_il, vbar, obar, g, D, BH, stream);
    }
    const bool big = m > 512;
#define BSA_RC(D_)                                                                                 \
    case D_:                                                                                       \
        return big ? launch_rank_coarse_t<D_, true>(qbar, kbar_il, vbar, obar, sel_idx, g, BH,     \
                                                    stream)                                        \
                   : launch_rank_coarse_t<D_, false>(qbar, kbar_il, vbar, obar, sel_idx, g, BH,    \
                                                     stream);
    switch (D) {
        BSA_RC(32)
        BSA_RC(64)
        BSA_RC(128)
    }
#undef BSA_RC
    return hipErrorInvalidValue;
}

}  // namespace bsa
