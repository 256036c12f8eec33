// Block-sparse attention forward for every shape the specialised kernels do not
// cover, on the gfx950 matrix cores: fp32 and bf16, head dim 32, 64 or 128, any
// tile of up to 1024 tokens.
//
// Every token of query block i attends, in one softmax, to the tokens of block
// i and of its n selected blocks (fine-grained attention equation plus the
// local block).  A wavefront owns 32 query rows (fp32: 16); a workgroup of up to 8
// wavefronts owns up to 256 (128) rows of one query block, whose wavefronts attend to
// the same keys.  The attended keys are walked as one flat sequence
// (bsa_flat_rows.h) in tiles of 64 (bf16) or 32 (fp32) keys that the workgroup
// shares through LDS: gathered with direct-to-LDS loads, double buffered, one
// barrier per tile.
//
// Transposed products as in the specialised kernels: S^T = K Q^T and
// O^T = V^T P^T, so that a lane holds one query column, the softmax reductions are
// in-register, and the S^T accumulator registers are the B operand of the second
// product.
//   fp32: v_mfma_f32_16x16x4_f32, i.e. fp32 products and sums throughout.  Lane
//         part p (of 4) supplies channels 16 j + 4 p + 0..3 of its row, so a 16-byte
//         read feeds four instructions; accumulator register r of 16 keys is, as it is,
//         the B operand of the keys 4 p + r.  With 16 rows to a wavefront instead of 32
//         the four that share a block of 64 cover each other's dependent products: 1.5
//         degrees, 8 heads, 385 -> 317 us (matrix pipe busy 62 -> 79 %), the 32 x 64
//         grid 18.2 -> 12.7 us.
//   bf16: v_mfma_f32_32x32x16_bf16.  The weights enter the second product as two
//         bf16 terms (16 significant bits): these shapes have always had their
//         weights multiplied in fp32, and keep that precision.  The last wavefront of a
//         block with at most 16 rows left takes the 16-wide form (Rows16): 12 x 24 tiles, 16
//         slices, 9 blocks, forward in us, head dim 32 tiles of 10 x 10 147 -> 137, 6 x 8
//         51 -> 45, 10 x 13 (five wavefronts) 321 -> 272; 64: 221 -> 217, 81 -> 75, 529 ->
//         475; backward at 64: 736 -> 721, 255 -> 243, 1,573 -> 1,386.
// Measured against the vector-ALU kernel that it replaces (one lane per query
// row, keys broadcast from LDS), select + forward: 131,072 tokens, 16 heads, head
// dim 32, bf16, 17 blocks of 128: 9.77 -> 1.25 ms; the 32 x 64 grid in fp32: 121
// -> 25 us (both with the selection as it is now).
// Softmax without a row maximum per tile: weights are taken against a reference
// that only moves when a row sum of a tile leaves the safe range.  The reference is
// the rounded product of a score and c2, and exp2(fma(s, c2, -m_ref)) sees what the
// rounding dropped: nothing that matters below kPlainRef, but more than the whole
// range of exp2 once scores reach 2^31 (masks by a large finite score).  From
// kPlainRef on a row keeps that remainder, and its weights are taken from
// (s c2 - m_ref) - m_rest, which is exactly 0 at the largest score, in the branch
// that moves references; rows below never leave the plain form.
#include "bsa_device.h"
#include "bsa_flat_rows.h"
#include "bsa_launch.h"
#include "bsa_mfma_common.h"

namespace bsa {

// References below this size are rounded by at most 2^-5: all weights of the row are
// off by the same factor of at most 2^(1/32), which the normalisation takes out.
constexpr float kPlainRef = 1048576.0f;

// NL: wavefronts that issue the gathers (1, 2 or 4; the workgroup has at least
// that many, up to 8).  row_chunks workgroups share a query block's rows,
// chunk_rows each.
// SPLIT > 1: as many groups of one or two (NL) wavefronts own the same rows and take
// the key tiles in turn, with tiles and a softmax of their own; the first group merges them
// at the end.  For launches that leave the chip idle; see key_split.
template <typename T, int D, int NL, int SPLIT, bool MIXED = false>
__global__ __launch_bounds__(SPLIT > 1 ? 64 * SPLIT * NL : NL == 4 ? 512 : NL == 2 ? 192 : 64,
                             SPLIT > 1 || NL == 1 || (NL == 2 && D == 128) ? 1
                             : D == 32 || (sizeof(T) == 4 && D == 128) ? 4 : 2)
void fwd_generic_kernel(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                        BSA_FWD_JOB_PARAMS(T), Geom g, uint32_t n_units, int row_chunks, int chunk_rows)
{
    // this workgroup's job, and its number inside the job
    const bool second_job = blockIdx.x >= jobs.n_first;
    const uint32_t wg = second_job ? blockIdx.x - jobs.n_first : blockIdx.x;
    const int32_t* __restrict__ sel_idx = second_job ? lists1 : lists0;
    T* __restrict__ out = second_job ? out1 : out0;
    float* __restrict__ lse = second_job ? lse1 : lse0;
    g.n_select = jobs.n_select[second_job ? 1 : 0];
    g.list_only = jobs.list_only[second_job ? 1 : 0];
    using Tile = FlatTile<T, D>;
    constexpr int KT = Tile::KT;
    __shared__ __attribute__((aligned(1024))) unsigned char k_lds[SPLIT][2][Tile::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_lds[SPLIT][2][Tile::TILE_BYTES];
    extern __shared__ __attribute__((aligned(16))) uint32_t tables_s[];

    const int lane = threadIdx.x & 63;
    const int waves = SPLIT == 1 ? 0 : (int)(blockDim.x >> 6) / SPLIT;       // of a group
    const int wg_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = SPLIT == 1 ? 0 : wg_wave / waves, wave = wg_wave - group * waves;
    const int b = g.block_tokens;

    int item;
    int64_t bh_idx;
    map_workgroup(g, wg, (uint32_t)row_chunks, n_units, bh_idx, item);
    const int i = item / row_chunks;
    const int row0 = (item - i * row_chunks) * chunk_rows;
    const int64_t base = bh_idx * g.n_tokens * D;
    const int64_t kv_base = kv_slice_of(g, bh_idx) * g.n_tokens * D;
    AttendedKeys<T, D, NL, SPLIT> keys;
    keys.init(g, sel_idx, bh_idx, i, tables_s, lane, wave, group);
    const int first_row = row0 + WaveTile<T>::ROWS * wave, end_row = min(b, row0 + chunk_rows);

    with_rows<T, MIXED>(end_row - first_row, [&](auto piece_key) {
    using K = typename decltype(piece_key)::type;
    using W = WaveTile<K>;
    const int col = lane & (W::ROWS - 1), part = lane / W::ROWS;
    TileReader<K, D> rd;
    rd.init(lane);
    // this wavefront's query rows
    const int tau_q = first_row + col;
    const bool valid = tau_q < end_row;
    const int64_t q_tok = token_of(g, i, valid ? tau_q : 0);
    typename RowPieces<K, D>::type qf[RowPieces<K, D>::N];
#pragma unroll
    for (int s = 0; s < RowPieces<K, D>::N; ++s) load_row<K>(q + base + q_tok * D, qf[s], s, part);
    __syncthreads();                                 // tables

    const int64_t slice_bytes = g.n_tokens * Tile::ROW_BYTES;
    const RowSource ks(k + kv_base, slice_bytes), vs(v + kv_base, slice_bytes);
    const uint32_t k_dst = lds_address(k_lds[group]), v_dst = lds_address(v_lds[group]);
    if (wave < NL) {
        keys.look_up();
        if (SPLIT == 1 || group < keys.tiles) keys.gather_next(ks, vs, k_dst, v_dst);
    }

    const float c2 = g.scale * 1.4426950408889634f;
    Column<K, D> oacc;
    clear_column<K, D>(oacc);
    float m_ref = -INFINITY, m_rest = 0.0f, l_run = 0.0f;
    uint64_t rests = 0;                              // lanes whose m_rest is not 0

    for (int c0 = 0; c0 < keys.tiles; c0 += SPLIT) {
        // tile c has landed and everyone is done with the other buffer
        wait_gathers();
        __syncthreads();
        const int c = c0 + group;
        if (SPLIT > 1 && c >= keys.tiles) continue;       // (the last round)
        const int buf = c0 / SPLIT & 1, other = (buf ^ 1) * Tile::TILE_BYTES;
        if (wave < NL && c + SPLIT < keys.tiles) keys.gather_next(ks, vs, k_dst + other, v_dst + other);
        const uint32_t at = (uint32_t)buf * Tile::TILE_BYTES;
#pragma unroll
        for (int hh = 0; hh < KT / 32; ++hh) {
            typename W::vec s = dot_tile<K, D>(rd, k_dst + at, 32 * hh * Tile::ROW_BYTES, qf, constant_tile<K>(0.0f));
            const int left = keys.total - (KT * c + 32 * hh);     // keys from this half tile on
            if (left < 32) {
                if (left <= 0) break;
#pragma unroll
                for (int r = 0; r < W::NR; ++r)
                    if (past_end<K>(r, part, left)) s[r] = -INFINITY;
            }
            ColumnPieces<K, D> v0;
            read_columns(rd, v_dst + at, 32 * hh * Tile::ROW_BYTES, 0, v0);
            typename W::vec p;
            float rs0 = 0.0f, rs1 = 0.0f;
#pragma unroll
            for (int r = 0; r < W::NR; r += 2) {
                p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -m_ref));
                p[r + 1] = __builtin_amdgcn_exp2f(fmaf(s[r + 1], c2, -m_ref));
                rs0 += p[r];
                rs1 += p[r + 1];
            }
            float rs = rs0 + rs1;
            if (__builtin_expect((__builtin_amdgcn_ballot_w64(!(rs <= kSumLimit)) | rests) != 0,
                                 0)) {
                // new reference from the row maxima; rescale what is there
                float mx = s[0];
#pragma unroll
                for (int r = 1; r < W::NR; ++r) mx = fmaxf(mx, s[r]);
                mx = column_max<K>(mx);
                const bool up = fmaf(mx, c2, -m_ref) > m_rest;
                const float m_new = up ? mx * c2 : m_ref;
                // no reference yet: all scores so far are below the range of fp32 once
                // multiplied with c2.  Their weights are exp2 of that product, i.e. 0;
                // NaN stays NaN
                const bool none = m_new == -INFINITY;
                const float neg_m = none ? 0.0f : -m_new;
                const float rest_new =
                    !up ? m_rest : !none && fabsf(m_new) >= kPlainRef ? fmaf(mx, c2, neg_m) : 0.0f;
                const float alpha =
                    none ? 1.0f : __builtin_amdgcn_exp2f((m_ref - m_new) + (m_rest - rest_new));
                m_ref = m_new;
                m_rest = rest_new;
                rests = __builtin_amdgcn_ballot_w64(rest_new != 0.0f);
                l_run *= alpha;
                scale_column<K, D>(oacc, alpha);
                rs = 0.0f;
#pragma unroll
                for (int r = 0; r < W::NR; ++r) {
                    p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, neg_m) - rest_new);
                    rs += p[r];
                }
            }
            l_run += rs;
            weighted_rows(rd, v_dst + at, 32 * hh * Tile::ROW_BYTES, v0, p, oacc);
        }
    }

    if constexpr (SPLIT > 1) {
        // groups 1 .. hand over what they have, lane by lane; the first group adds it up
        constexpr int VALUES = (int)sizeof(Column<K, D>) / 4 + 3;
        static_assert((SPLIT - 1) * NL * VALUES * 256 <= SPLIT * 2 * Tile::TILE_BYTES * 2,
                      "fits the tiles");
        constexpr int HALF = SPLIT * 2 * Tile::TILE_BYTES / 256;       // values per array and lane
        auto place = [&](int of_group, int value) -> float* {
            const int at = ((of_group - 1) * waves + wave) * VALUES + value;
            return (at < HALF ? (float*)k_lds + at * 64 : (float*)v_lds + (at - HALF) * 64) + lane;
        };
        __syncthreads();
        if (group > 0) {
            *place(group, 0) = m_ref;
            *place(group, 1) = m_rest;
            *place(group, 2) = l_run;
            int at = 3;
#pragma unroll
            for (auto& a : oacc.a)
#pragma unroll
                for (int r = 0; r < (int)sizeof(a) / 4; ++r) *place(group, at++) = a[r];
        }
        __syncthreads();
        if (group > 0) return;
        for (int from = 1; from < SPLIT; ++from) {
            const float m = *place(from, 0), rest = *place(from, 1), l = *place(from, 2);
            const bool up = m > m_ref || (m == m_ref && rest > m_rest);
            const float m_new = up ? m : m_ref, rest_new = up ? rest : m_rest;
            const bool none = m_new == -INFINITY;
            const float old = none ? 1.0f : __builtin_amdgcn_exp2f((m_ref - m_new) + (m_rest - rest_new));
            const float add = none ? 1.0f : __builtin_amdgcn_exp2f((m - m_new) + (rest - rest_new));
            m_ref = m_new;
            m_rest = rest_new;
            l_run = l_run * old + l * add;
            int at = 3;
#pragma unroll
            for (auto& a : oacc.a)
#pragma unroll
                for (int r = 0; r < (int)sizeof(a) / 4; ++r) a[r] = a[r] * old + *place(from, at++) * add;
        }
    }

    const float l_tot = column_sum<K>(l_run);
    if (valid) {
        const float inv_l = 1.0f / l_tot;
        store_column<D>(out + base + q_tok * D, oacc, inv_l, nullptr, 0.0f, part);
        if (lse && part == 0)
            lse[bh_idx * g.n_tokens + q_tok] =
                (m_ref + (m_rest + __builtin_amdgcn_logf(l_tot))) * 0.6931471805599453f;
    }
    });
}

// Row wavefronts of a workgroup at most, and groups that share its keys, for a launch of
// `wavefronts` row wavefronts, which take `pairs` workgroups when two share one where a block
// has two, and `tiles` key tiles each.  What bounds a small launch is the chain of one
// wavefront through its tiles while most CUs are idle; what a split costs is two barriers
// and the merge, 0.5 to 2 us.
// 1 x 4: a workgroup per row wavefront, four groups (a wavefront per SIMD of its CU).
// 2 x 2: pairs, two groups.  us, unsplit | 1 x 4 | 2 x 2, tiles of 32 (fp32) or 64 keys:
//   * up to 256 wavefronts, fp32, blocks of 16, head dim 32: 1 tile 4.8 | 5.9 | 5.3, 2 tiles
//     5.7 | 6.1 | 5.5, 3 6.6 | 6.2 | 6.3, 8 11.2 | 7.6 | 8.5; 64: 1 5.9 | 7.4 | 6.6, 2 7.4 |
//     7.8 | 6.8, 3 9.0 | 7.8 | 8.4, 8 16.9 | 10.1 | 11.7.  bf16, blocks of 36, head dim 64: 1
//     5.4 | 8.2 | 6.4, 3 8.2 | 8.8 | 8.1, 4 9.5 | 9.0 | 8.3, 6 11.9 | 10.5 | 9.6, 8 14.6 |
//     10.9 | 11.0.
//   * up to 512 in at most 256 pairs: as the pairs above (bf16 head dim 64, 480 wavefronts,
//     4 tiles 9.5 | - | 8.4; 128, 6 tiles 17.3 | - | 14.2).
//   * more workgroups than CUs (blocks of one row wavefront, or three).  Head dim 128: the
//     tiles of two groups take 128 KiB of LDS, so that these run in two rounds, where
//     unsplit ones fit a CU twice: never (368 wavefronts, fp32, 8 tiles 29.5 | - | 35.1, bf16,
//     4 15.5 | - | 23.2).  64: single wavefronts as above (fp32, 368, 2 tiles 7.9 | - | 7.3, 8
//     17.3 | - | 12.7; bf16, 4 10.6 | - | 9.6), three not (fp32, 480, 4 tiles 9.8 | - | 10.3).
//     32: from 8 tiles (fp32, 368, 4 tiles 7.8 | - | 8.1, 8 11.5 | - | 11.2).
// 1,024 wavefronts: head dim 64, 10 tiles 19.4 | 39.1 | 18.8, 128 31.4 | - | 38.0.
struct KeySplit {
    int max_waves, groups;
};
template <typename T, int D>
static KeySplit key_split(int64_t wavefronts, int64_t pairs, bool single, int64_t tiles, int most)
{
    // tiles from which two groups and four pay
    const int two = sizeof(T) == 4 ? 2 : 4, four = sizeof(T) == 4 ? 3 : 7;
    if (wavefronts <= 256 && D < 128 && tiles >= four) return {1, 4};
    const bool pays = pairs <= 256 || (D == 64 && single) ? tiles >= two : D == 32 && tiles >= 8;
    if (wavefronts <= 512 && pays) return {2, 2};
    return {most, 1};
}

template <typename T, int D, int SPLIT, bool MIXED = false>
static auto kernel_of(int waves)
{
    if constexpr (SPLIT == 4) {                       // (head dim 128: not chosen)
        return fwd_generic_kernel<T, D, 1, D == 128 ? 2 : 4>;
    } else if constexpr (SPLIT == 2) {
        return waves >= 2 ? fwd_generic_kernel<T, D, 2, 2> : fwd_generic_kernel<T, D, 1, 2>;
    } else {
        return waves >= 4 ? fwd_generic_kernel<T, D, 4, 1, MIXED>
               : waves >= 2 ? fwd_generic_kernel<T, D, 2, 1, MIXED>
                            : fwd_generic_kernel<T, D, 1, 1, MIXED>;
    }
}

template <typename T, int D>
static hipError_t launch_t(const void* q, const void* k, const void* v, const FwdJob* jobs,
                           int n_jobs, const Geom& g, int64_t BH, hipStream_t stream)
{
    // fp32, head dim 32: with 8 wavefronts, of 16 rows, the last of an odd number of them
    // leaves SIMDs uneven (10 x 10 tiles 589 us, with 4 568, with 32-row wavefronts 560;
    // 16 x 16 1,168 against 1,170).  At head dim 128 four wavefronts per SIMD need 128
    // registers (5 spill outside of the tile loop): blocks of 256 4.37 -> 4.10 ms.
    const int most = sizeof(T) == 4 && D == 32 ? 4 : 8;
    const RowSplit whole(g.block_tokens, most, WaveTile<T>::ROWS);
    int listed = 0;
    int64_t keys = 0;                                 // of the job with most
    for (int j = 0; j < n_jobs; ++j) {
        listed = jobs[j].n_select + 1 > listed ? jobs[j].n_select + 1 : listed;
        const int64_t attended =
            (int64_t)(jobs[j].n_select + 1 - jobs[j].list_only) * g.block_tokens;
        keys = attended > keys ? attended : keys;
    }
    constexpr int KT = FlatTile<T, D>::KT;
    const int64_t blocks = BH * g.n_blocks * n_jobs;
    const RowSplit pairs(g.block_tokens, 2, WaveTile<T>::ROWS);
    const KeySplit ks = key_split<T, D>(blocks * whole.chunks * whole.waves, blocks * pairs.chunks,
                                        pairs.waves == 1, (keys + KT - 1) / KT, most);
    const RowSplit rows(g.block_tokens, ks.max_waves, WaveTile<T>::ROWS);
    const int nw = rows.waves, split = ks.groups;
    const int64_t wgs = (int64_t)g.kv_group * g.n_blocks * rows.chunks;    // per key/value slice
    auto kernel = split == 4 ? kernel_of<T, D, 4>(nw)
                  : split == 2 ? kernel_of<T, D, 2>(nw)
                  : rows.narrow ? kernel_of<T, D, 1, sizeof(T) == 2>(nw) : kernel_of<T, D, 1>(nw);
    return launch_slices(BH / g.kv_group, wgs * 64 * nw * split, [&](int64_t first, int64_t slices) {
        const int64_t row = first * g.kv_group * g.n_tokens, kv = first * g.n_tokens * D;
        FwdJob piece[2];
        for (int j = 0; j < n_jobs; ++j) {
            piece[j] = jobs[j];
            piece[j].lists += first * g.kv_group * g.n_blocks * jobs[j].n_select;
            piece[j].out = (T*)jobs[j].out + row * D;
            if (jobs[j].lse) piece[j].lse += row;
        }
        return launch_jobs(piece, n_jobs, slices * wgs, 64 * nw * split,
                           [&](const FwdJob& a, const FwdJob& b, const FwdShape& j, unsigned grid) {
                               kernel<<<dim3(grid), dim3(64 * nw * split), flat_table_bytes(g, listed, split),
                                        stream>>>((const T*)q + row * D, (const T*)k + kv,
                                                  (const T*)v + kv, a.lists, b.lists, (T*)a.out,
                                                  (T*)b.out, a.lse, b.lse, j, g, (uint32_t)slices,
                                                  rows.chunks, WaveTile<T>::ROWS * nw);
                           });
    });
}

hipError_t launch_fwd_generic(bool is_bf16, const void* q, const void* k, const void* v,
                              const FwdJob* jobs, int n_jobs, const Geom& g, int D, int64_t BH,
                              hipStream_t stream)
{
#define BSA_CASE(DD)                                                                    \
    case DD:                                                                            \
        return is_bf16 ? launch_t<uint16_t, DD>(q, k, v, jobs, n_jobs, g, BH, stream)   \
                       : launch_t<float, DD>(q, k, v, jobs, n_jobs, g, BH, stream);
    switch (D) {
        BSA_CASE(32)
        BSA_CASE(64)
        BSA_CASE(128)
    }
#undef BSA_CASE
    return hipErrorInvalidValue;
}

}  // namespace bsa
