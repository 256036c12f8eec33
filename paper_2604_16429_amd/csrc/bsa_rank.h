// Scores and top-n of many key blocks (gfx950): 32 query blocks per workgroup, scores on
// the fp32 matrix cores, the best n of each row kept in a short list while they stream by.
//
// A score is the chain acc = fma(qbar[d], kbar[d], acc), d ascending from +0, bit for bit:
// v_mfma_f32_32x32x1_2b_f32 does one fused multiply-add per output element (the other
// matrix instructions sum several products in an order of their own), so a chain of D of
// them is that chain for 64 keys x 32 queries.
//
// What bounds select_block (bsa_select.hip) with many blocks is L2: rows of m scores fill
// LDS, so that a workgroup holds four query blocks and reads all pooled keys for them, 12 GB
// for 16 slices of 3,422 blocks.  Here a workgroup reads them for 32, and only candidates go
// to LDS.  Selection, us, select_block | here: 0.25 degrees (16 slices of 4,050 blocks, head
// dim 64, pooling 770 of it) 1,605 | 920; 16 of 3,422 (8 x 16 tiles) 999 | 607; 24 of
// 2,276, head dim 128, 1,194 | 774.  A step of 256 keys takes 5,200 cycles of matrix
// instructions at head dim 64 and 6,000 for the candidates (mask 1,100, lists 2,000, pruning
// and waiting 3,000).  Entering the candidates of a step between the matrix instructions of
// the next was slower (717 against 624 us, 4,050 blocks x 16, head dim 64, then): the
// branches, and the code of both copies.
#pragma once

#include "bsa_device.h"

namespace bsa {

// Order-preserving map fp32 -> u32 (larger float <=> larger integer).  Every
// non-NaN input maps to a value >= 0x007fffff; the clamp keeps even a NaN bit
// pattern away from 0, which marks "removed".
__device__ __forceinline__ uint32_t rank_key(float s)
{
    const uint32_t u = __float_as_uint(s + 0.0f);    // -0 -> +0
    return max((u & 0x80000000u) ? ~u : (u | 0x80000000u), 1u);
}

// Position of this lane among the set lanes of mask.
__device__ __forceinline__ int place_in(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

typedef __attribute__((ext_vector_type(32))) float f32x32;

constexpr int kRankRows = 32;       // query blocks per workgroup
constexpr int kRankList = 96;       // entries of a row's list
constexpr int kRankPicks = 32;      // blocks picked at most
constexpr int kRankMost = 48;       // entries of a list that is ranked, at most

// A row's list holds candidates as composites (key << 32 | ~j), which are distinct and order
// exactly as the ranking does.  Candidates that n entries of the list are known to beat
// are not entered: those with key < floor_key, and of key == floor_key those with
// j >= floor_j.  limit: where an entry did not fit any more.
struct RankLists {
    uint64_t entry[kRankRows][kRankList + 1];        // (+ 1: rows on different LDS banks)
    uint32_t count[kRankRows], limit[kRankRows], floor_key[kRankRows];
    int32_t floor_j[kRankRows];
    int32_t again[2];
};

// Sums over the eight lanes 8 i .. 8 i + 7.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_shifted(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t sum8(uint32_t v)
{
    v += dpp_shifted<0xB1>(v);                       // quad_perm [1,0,3,2]
    v += dpp_shifted<0x4E>(v);                       // quad_perm [2,3,0,1]
    return v + dpp_shifted<0x141>(v);                // row_half_mirror
}
__device__ __forceinline__ uint32_t max8(uint32_t v)
{
    v = max(v, dpp_shifted<0xB1>(v));
    v = max(v, dpp_shifted<0x4E>(v));
    return max(v, dpp_shifted<0x141>(v));
}

// If one of the lists of rows row0 .. row0 + 7 holds more than `more` entries, shortens all
// that hold more than `most` to between n and `most` of their best and sets their floors.
// One wavefront, eight lanes to a row.  The threshold is found bit by bit, first of the keys, then, where too many
// entries have the last key, of their block indices.
__device__ __forceinline__ void prune_lists(RankLists& s, int row0, int n, int more, int most, int lane)
{
    const int sub = lane & 7, row = row0 + (lane >> 3);
    const int valid = (int)min(min(s.count[row], s.limit[row]), (uint32_t)kRankList);
    if (__builtin_amdgcn_ballot_w64((int)s.count[row] > more) == 0) return;
    const bool active = valid > most;
    uint64_t* const list = s.entry[row];
    constexpr int PER = kRankList / 8;
    uint32_t high[PER], top = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        high[i] = 8 * i + sub < valid ? (uint32_t)(list[8 * i + sub] >> 32) : 0u;
        top = max(top, high[i]);
    }
    top = max8(top);
    // every entry lies between the floor and the largest: their common upper bits are known
    const uint32_t differ = top ^ s.floor_key[row];
    int bits = active ? 32 - __builtin_clz(differ | 1u) : 0;
    uint32_t t = active ? (bits < 32 ? top >> bits << bits : 0u) : 0u;
    int have = active ? valid : most;
    while (__builtin_amdgcn_ballot_w64(have > most && bits > 0)) {
        const bool going = have > most && bits > 0;
        --bits;
        const uint32_t up = t | (going ? 1u << (bits & 31) : 0u);
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) c += high[i] >= up ? 1u : 0u;
        c = sum8(c);
        if (going && (int)c >= n) { t = up; have = (int)c; }
    }
    uint32_t u = 0;                                  // of the entries with key t: lowest low word
    const bool ties = have > most;
    if (__builtin_amdgcn_ballot_w64(ties)) {
        uint32_t low[PER], above = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            above += high[i] > t ? 1u : 0u;
            low[i] = high[i] == t && 8 * i + sub < valid ? (uint32_t)list[8 * i + sub] : 0u;
        }
        above = sum8(above);
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t up = u | 1u << bit;
            uint32_t c = 0;
#pragma unroll
            for (int i = 0; i < PER; ++i) c += low[i] >= up ? 1u : 0u;
            if ((int)(above + sum8(c)) >= n) u = up;
        }
        if (!ties) u = 0;
    }
    // what stays moves to the front, eight entries at a time (never past what was read)
    int at = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint64_t e = list[8 * i + sub];
        const bool keep = active && 8 * i + sub < valid &&
                          (high[i] > t || (high[i] == t && (uint32_t)e >= u));
        const uint32_t kept = (uint32_t)(__builtin_amdgcn_ballot_w64(keep) >> (lane & 56)) & 255u;
        if (keep) list[at + __builtin_popcount(kept & ((1u << sub) - 1u))] = e;
        at += __builtin_popcount(kept);
    }
    if (active && sub == 0) {
        s.count[row] = (uint32_t)at;
        s.limit[row] = kRankList;
        s.floor_key[row] = t;
        s.floor_j[row] = ties ? (int32_t)~u : 0x7fffffff;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// K-th largest of a lane's 32 scores (or a smaller one, where some are equal), as its key.
template <int K>
__device__ __forceinline__ uint32_t lane_kth(const f32x32& score, uint32_t removed)
{
    uint32_t best[K];
#pragma unroll
    for (int i = 0; i < K; ++i) best[i] = 0;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const uint32_t key = removed >> (31 - e) & 1u ? 0u : rank_key(score[e]);
#pragma unroll
        for (int i = K - 1; i > 0; --i) best[i] = max(best[i], min(best[i - 1], key));
        best[0] = max(best[0], key);
    }
    return best[K - 1];
}

// LDS of a workgroup: the lists, the pooled queries as [D/4][32 rows] of 4 channels, and
// each wavefront's scores, 16 of 32 at a time: [4][lane] of 4.
template <int D> struct RankShared {
    RankLists lists;
    float4 q[D / 4][kRankRows];
    float4 stage[4][4][64];
};

// A workgroup barrier that waits for LDS accesses only (loads of keys stay in flight).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One workgroup of 256 threads ranks 32 consecutive query blocks of one (batch, head); m >=
// 256, 1 <= n <= 32.  Its four wavefronts share the rows: keys come in groups of 64,
// wavefront w takes the groups 4 s + w in an order spread over all of them (stride, coprime
// to their number: the first groups then are a sample and the floor is soon close to its
// last value, also where scores rise along the grid).  Lane l has query l % 32 and, of
// a group, keys 8 i + 4 (l / 32) + 0..3.  After each step rows with long lists are pruned.
template <int D>
__device__ __forceinline__ void rank_block(const float* __restrict__ qbar,
                                           const float* __restrict__ kbar_il,
                                           int32_t* __restrict__ sel_idx, const Geom& g, int stride,
                                           uint32_t vblock, RankShared<D>& shared)
{
    constexpr int CH = D == 128 ? 64 : 32, QUADS = D / 4;        // channels read ahead
    RankLists& s = shared.lists;
    const int m = g.n_blocks, n = g.n_select;
    const int row_groups = (m + kRankRows - 1) / kRankRows;
    const int64_t bh_idx = vblock / (uint32_t)row_groups;
    const int i0 = (int)(vblock - (uint32_t)bh_idx * (uint32_t)row_groups) * kRankRows;
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool row_valid = i0 + col < m;
    const float4* const keys = (const float4*)(kbar_il + kv_slice_of(g, bh_idx) * m * D);   // [D/4][m]
    float* const stage = (float*)shared.stage[wave];

    const int steps = (m + 255) / 256;               // of four groups
    const int most = n + kRankMost - kRankPicks;     // entries of a list that was pruned
    auto first_of = [&](int at) { return 64 * (4 * at + wave); };
    float4 next[CH / 4];
    auto load = [&](int c, int j) { return keys[(int64_t)c * m + j]; };
    int at = 0;                                      // groups 4 at + 0..3 are next
    {
        const int j = min(first_of(at) + lane, m - 1);
#pragma unroll
        for (int c = 0; c < CH / 4; ++c) next[c] = load(c, j);
    }
    for (int e = threadIdx.x; e < QUADS * kRankRows; e += 256) {
        const int row = e % kRankRows, c = e / kRankRows;
        shared.q[c][row] = *(const float4*)(qbar + (bh_idx * m + min(i0 + row, m - 1)) * D + 4 * c);
    }
    if (threadIdx.x < kRankRows) {
        s.count[threadIdx.x] = 0;
        s.limit[threadIdx.x] = kRankList;
        s.floor_key[threadIdx.x] = 0xffffffffu;
        s.floor_j[threadIdx.x] = 0x7fffffff;
    }
    if (threadIdx.x < 2) s.again[threadIdx.x] = 0;
    __syncthreads();

    int turn = 0;
    for (int step = 0; step < steps; ++step) {
        const int base = first_of(at), this_lane = min(base + lane, m - 1);
        at += stride;
        if (at >= steps) at -= steps;
        const int next_lane = min(first_of(at) + lane, m - 1);    // (a group in range, used or not)
        f32x32 acc;
#pragma unroll
        for (int e = 0; e < 32; ++e) acc[e] = 0.0f;
        float4 q = shared.q[0][col];
#pragma unroll
        for (int c = 0; c < QUADS; ++c) {
            const float4 k4 = next[c % (CH / 4)], q4 = q;
            if (c + 1 < QUADS) q = shared.q[c + 1][col];
            next[c % (CH / 4)] = c + CH / 4 < QUADS ? load(c + CH / 4, this_lane)
                                                    : load(c + CH / 4 - QUADS, next_lane);
            acc = __builtin_amdgcn_mfma_f32_32x32x1f32(k4.x, q4.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x1f32(k4.y, q4.y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x1f32(k4.z, q4.z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x1f32(k4.w, q4.w, acc, 0, 0, 0);
        }
        // element e: key block base + 32 (e / 16) + 8 (e % 16 / 4) + 4 half + e % 4; bit
        // 31 - e of a mask.  Removed: the query block itself and blocks past the end.
        auto j_of = [&](int e) { return base + 32 * (e >> 4) + 8 * ((e & 15) >> 2) + 4 * half + (e & 3); };
        const bool has_own = !g.own_is_candidate && base < i0 + kRankRows && base + 64 > i0;
        uint32_t removed = row_valid ? 0u : ~0u;
        if (has_own || base + 64 > m) {
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                const int j = j_of(e);
                removed |= j >= m || (has_own && j == i0 + col) ? 1u << (31 - e) : 0u;
            }
        }
        if (step == 0) {
            // all eight lanes of a row have K keys that reach the smallest of their K-th
            // largest: with 8 K >= n a floor for a start (every wavefront has 64 keys)
            const uint32_t kth = n <= 8 ? lane_kth<1>(acc, removed) : n <= 16 ? lane_kth<2>(acc, removed)
                                                                     : lane_kth<4>(acc, removed);
            if (row_valid) atomicMin(&s.floor_key[col], kth);
            lds_barrier();
        }
        // enter what reaches the floor; a lane whose candidates do not fit tries again after
        // the lists have been pruned (the first 32 of a list that was pruned do fit)
        bool pending = true;
        for (;;) {
            // key > above in terms of the scores (above 0: any; NaN is entered and ranked by
            // its key; -0 counts as +0, so that its lower neighbour is -0's)
            const uint32_t floor_key = s.floor_key[col];
            uint32_t above = floor_key == 0 ? 0u : floor_key - (base < s.floor_j[col] ? 1u : 0u);
            above -= above == 0x7fffffffu ? 1u : 0u;
            const float floor = __uint_as_float(above & 0x80000000u ? above ^ 0x80000000u : ~above);
            uint32_t mask = 0;
#pragma unroll
            for (int e = 0; e < 32; ++e) mask = mask + mask + (acc[e] <= floor ? 0u : 1u);
            mask = pending ? mask & ~removed : 0u;
            const int mine = __builtin_popcount(mask);
            const int first = mine > 0 ? (int)atomicAdd(&s.count[col], (uint32_t)mine) : 0;
            const bool fits = first + mine <= kRankList;
            if (!fits) atomicMin(&s.limit[col], (uint32_t)first);
            pending = !fits;
            if (!fits) mask = 0u;
            uint64_t* to = &s.entry[col][first];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t part = h == 0 ? mask & 0xffff0000u : mask << 16;
                if (__builtin_amdgcn_ballot_w64(part != 0u) == 0) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *(float4*)(stage + (64 * i + lane) * 4) =
                        make_float4(acc[16 * h + 4 * i], acc[16 * h + 4 * i + 1],
                                    acc[16 * h + 4 * i + 2], acc[16 * h + 4 * i + 3]);
                while (part != 0u) {
                    const int e = __builtin_clz(part);
                    part &= ~(0x80000000u >> e);
                    const uint32_t key = rank_key(stage[(64 * (e >> 2) + lane) * 4 + (e & 3)]);
                    *to++ = (uint64_t)key << 32 | (uint32_t)~(j_of(e) + 32 * h);
                }
            }
            lds_barrier();
            const uint32_t count = s.count[8 * wave + (lane & 7)];
            if (__builtin_amdgcn_ballot_w64(count > kRankList) && lane == 0) s.again[turn & 1] = 1;
            prune_lists(s, 8 * wave, n, step + 1 == steps ? kRankMost : kRankList - 32, most, lane);
            if (threadIdx.x == 0) s.again[(turn & 1) ^ 1] = 0;
            lds_barrier();
            const bool again = s.again[turn & 1] != 0;
            ++turn;
            if (!again) break;
        }
    }

    // the n best are among the up to kRankMost entries of a list: place each by counting the larger
    const int n_rows = min(kRankRows, m - i0);
    for (int r = 8 * wave; r < 8 * wave + 8 && r < n_rows; ++r) {
        const int count = __builtin_amdgcn_readfirstlane((int)min(s.count[r], (uint32_t)kRankMost));
        const uint64_t mine = lane < count ? s.entry[r][lane] : 0ull;
        int rank = 0;
        for (int t = 0; t < count; ++t) {
            const uint64_t c =
                ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine >> 32), t) << 32) |
                (uint32_t)__builtin_amdgcn_readlane((int)mine, t);
            rank += c > mine ? 1 : 0;
        }
        if (lane < count && rank < n)
            sel_idx[(bh_idx * m + i0 + r) * n + rank] = (int32_t)~(uint32_t)mine;
    }
}

}  // namespace bsa
