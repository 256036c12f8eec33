// Backward of the block-sparse attention on the gfx950 matrix cores (bf16 MFMA,
// fp32 accumulation), selection held fixed: no gradient flows through the
// top-n choice (Appendix "Block-sparse attention implementation").
//
// With P the attention weights of the forward pass, recomputed from the stored
// log-sum-exp as P = exp(scale * q.k - lse), and delta_l = dO_l . O_l:
//   dV_t = sum_l P_lt dO_l          dP_lt = dO_l . v_t
//   dS_lt = P_lt (dP_lt - delta_l)
//   dQ_l = scale * sum_t dS_lt k_t  dK_t = scale * sum_l dS_lt q_l
// where t runs over the keys of the blocks query block i attends to (itself and
// its selection) and l over the queries of the blocks that attend to t's block.
//
// Two main kernels, both built from 32 x 32 x 16 bf16 MFMAs on 64-token tiles that
// the wavefronts of a workgroup share through LDS (direct-to-LDS gathers,
// double buffered, one workgroup barrier per tile):
//   dq kernel    one workgroup per query block, a wavefront per 32 query rows,
//                walks the attended K/V sub-tiles like the forward pass.  Per
//                32-key tile: S^T = K Q^T and dP^T = V dO^T (a lane holds one
//                query column, so lse and delta are per-lane scalars),
//                dS^T in registers is the B operand of dQ^T += K^T dS^T, whose A
//                operand comes from the transposing LDS read of the K tile.
//   dk/dv kernel one workgroup per key/value block, a wavefront per 32 key rows
//                (their K and V rows stay in registers as B operands).  It
//                lists, in ascending order, the query blocks that attend to
//                its block (the paper's "query blocks connected to a key/value
//                block"), from a reverse map of the selection that a small
//                kernel builds first (bsa_bwd.hip): a bit matrix, one bit per
//                (key block, query block).  No floating-point atomics: the ascending list
//                fixes the summation order.  It then walks their Q/dO
//                sub-tiles.  Per 32-query tile: S = Q K^T and dP = dO V^T (rows
//                are queries now: lse and delta come from LDS per row), and
//                dV^T += dO^T P, dK^T += Q^T dS with the transposing LDS read
//                of the dO / Q tile.  One pass for both head dims: at 128, where
//                the accumulators take half of the registers, V stays in LDS.
// Waits for gathers are of the form that the compiler accounts for (wait_gathers):
// otherwise it waits, in front of the first use of the stationary rows inside the loop,
// for the loads that it issued before the loop, i.e. for the tile that was just
// requested.
// The difference dP - delta costs no vector instruction: the accumulator of dP
// starts from it (dq: 16 registers that hold the lane's -delta; dk/dv: delta as it is
// read from LDS, V negated in registers, so that -dS comes out and dK is scaled by
// -scale).  Vector and matrix instructions of a wavefront follow each other for a good
// part, so the 32 instructions per 32 x 32 tile count: select + forward + backward at
// 1.5 degrees, head dim 128, batch 4: 8.97 -> 8.79 ms; grouped heads at head dim 64,
// batch 12: 8.99 -> 8.84 ms.
#include <type_traits>

#include "bsa_device.h"
#include "bsa_launch.h"
#include "bsa_mfma_common.h"

namespace bsa {

namespace bwdm {

constexpr float kLog2e = 1.4426950408889634f;

// 16-byte chunk swizzle of an LDS row (8 or 16 chunks): a bijection of row % 8
// whose upper two bits differ over 4 aligned rows (row-fragment reads take the
// same chunk of 8 consecutive rows, transposing reads a chunk pair of 4 rows).
__device__ __forceinline__ int swz(int row, int chunk)
{
    return chunk ^ (((row & 3) << 1) | ((row >> 2) & 1));
}

// The gathers are the forms the compiler does not track: with the tracked ones
// it waited, in front of the first read of tile c, for the loads of tile c + 1
// (one array per double buffer), i.e. for a whole memory latency per tile that
// only the SIMD's other wavefront covered.  1.5 degree grid, head dim 64, grouped
// heads, batch 12: select + forward + backward 9.50 -> 9.39 ms; head dim 128,
// batch 4: 9.37 -> 9.17 ms.
//
// Geometry of 64-token x D tiles gathered into LDS by a workgroup of NW
// wavefronts.  A tile is SLABS loads of 1 KiB (RPS token rows each); wavefront
// w issues slabs w, w + NW, ...; lane l fills LDS chunk l of the slab, i.e. row
// l / LPR, swizzled chunk l % LPR, and therefore fetches the global chunk that
// swizzles to that slot.
template <int D, int NW>
struct TileIO {
    static constexpr int ROW_BYTES = D * 2;
    static constexpr int TILE_BYTES = 64 * ROW_BYTES;
    static constexpr int SLABS = TILE_BYTES / 1024;
    static constexpr int RPS = 1024 / ROW_BYTES;       // token rows per slab
    static constexpr int LPR = ROW_BYTES / 16;         // lanes per token row
    static constexpr int MINE = SLABS / NW;            // slabs per wavefront
    static_assert(SLABS % NW == 0, "slabs split evenly between wavefronts");

    uint32_t voff[MINE];        // byte offset of this lane's chunk inside a sub-tile
    uint32_t tok_off;           // byte offset (fp32 rows) of token `lane` of a sub-tile
    int wave;

    __device__ __forceinline__ void init(const Geom& g, int lane, int wave_)
    {
        wave = wave_;
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int slab = wave + j * NW;
            const int t = RPS * slab + lane / LPR;                    // token row 0..63
            voff[j] = (uint32_t)(sub_tile_pos(g, t) * ROW_BYTES + swz(t, lane % LPR) * 16);
        }
        tok_off = (uint32_t)(sub_tile_pos(g, lane) * 4);
    }
    // this wavefront's share of one tile (origin: byte offset of the sub-tile's
    // first token in a [N, D] bf16 slice)
    __device__ __forceinline__ void gather(i32x4 rsrc, uint32_t origin,
                                           unsigned char* lds_tile) const
    {
        const uint32_t dst = lds_address(lds_tile);
#pragma unroll
        for (int j = 0; j < MINE; ++j)
            load_lds_16(rsrc, voff[j], origin, dst + (uint32_t)(wave + j * NW) * 1024u);
    }
    // 64 fp32 values (one per token of the sub-tile) from a [N] fp32 slice;
    // origin_tok: index of the sub-tile's first token
    __device__ __forceinline__ void gather_f32(i32x4 rsrc, uint32_t origin_tok,
                                               float* lds_vec) const
    {
        load_lds_4(rsrc, tok_off, origin_tok * 4u, lds_address(lds_vec));
    }
};

// Row fragment: lane (l32, half) reads channels 16 ks + 8 half .. + 7 of tile
// row row0 + l32 (A operand "rows x channels", or B operand of the same shape).
template <int D>
__device__ __forceinline__ bf16x8 row_frag(const unsigned char* tile, int row0, int ks, int l32,
                                           int half)
{
    const int row = row0 + l32;
    return *(const bf16x8*)(tile + row * (D * 2) + swz(row, 2 * ks + half) * 16);
}

// Transposed fragment: A operand "channels 32 dt .. x tile rows row0 .. row0+15"
// through the transposing LDS read (source lane s of 16-lane group gq supplies
// 8 bytes of row row0 + 8 rd + 4 (gq/2) + s/4, channel 16 (gq%2) + 4 (s%4) + 32 dt).
template <int D>
__device__ __forceinline__ bf16x8 trans_frag(const unsigned char* tile, int row0, int dt,
                                             int lane)
{
    const int s16 = lane & 15, gq = lane >> 4;
    const int col = 16 * (gq & 1) + 4 * (s16 & 3) + 32 * dt;
    bf16x4 part[2];
#pragma unroll
    for (int rd = 0; rd < 2; ++rd) {
        const int row = row0 + 8 * rd + 4 * (gq >> 1) + (s16 >> 2);
        const unsigned char* src = tile + row * (D * 2) + swz(row, col >> 3) * 16 + (col & 7) * 2;
        part[rd] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, src));
    }
    return __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ f32x16 zero_tile()
{
    const f32x16 z = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f,
                      0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    return z;
}

// ---------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------
template <int D, int NW>
__device__ __forceinline__ void dq_body(const uint16_t* __restrict__ q,
                                        const uint16_t* __restrict__ k,
                                        const uint16_t* __restrict__ v,
                                        const uint16_t* __restrict__ dout,
                                        const float* __restrict__ lse2,
                                        const float* __restrict__ delta,
                                        const int32_t* __restrict__ sel_idx,
                                        uint16_t* __restrict__ dq, const Geom& g,
                                        uint32_t n_units)
{
    constexpr int KS = D / 16, DT = D / 32;
    using IO = TileIO<D, NW>;
    // [buffer][K tile, V tile]
    __shared__ __attribute__((aligned(4 * IO::TILE_BYTES))) unsigned char tiles_s[2][2][IO::TILE_BYTES];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int subs = g.block_tokens / 64;

    // workgroup -> (query slice, query block)
    int i;
    int64_t bh_idx;
    map_workgroup(g, blockIdx.x, 1, n_units, bh_idx, i);
    const int64_t base = bh_idx * g.n_tokens * D;
    const int64_t kv_base = kv_slice_of(g, bh_idx) * g.n_tokens * D;
    // The attended blocks: block i itself followed by its selected blocks, or,
    // in list-only mode, exactly the listed blocks.
    const int list_only = g.list_only;
    const int32_t* sel_row = sel_idx + (bh_idx * g.n_blocks + i) * g.n_select + list_only;
    const int first = list_only ? sel_row[-1] : i;
    const int n = g.n_select - list_only;        // blocks after the first
    const uint32_t slice_bytes = (uint32_t)(g.n_tokens * D * 2);
    const i32x4 k_rsrc = buffer_desc(k + kv_base, slice_bytes);
    const i32x4 v_rsrc = buffer_desc(v + kv_base, slice_bytes);

    IO io;
    io.init(g, lane, wave);
    auto origin_of = [&](int beta) -> uint32_t {     // byte offset of a block's first token
        const int br = beta / g.blocks_per_row, bc = beta - br * g.blocks_per_row;
        return (uint32_t)((br * g.block_h * g.grid_w + bc * g.block_w) * (D * 2));
    };
    const int pairs = (n + 1) * subs;
    // the listed blocks sit in the lanes of one register (up to 64 of them), so
    // that finding the next tile costs no memory access inside the loop
    const int sel_mine = (n <= 64 && lane < n) ? sel_row[lane] : 0;
    auto origin_of_pair = [&](int c) -> uint32_t {   // attended block c / subs, sub-tile c % subs
        const int cb = c / subs, ct = c - cb * subs;
        const int beta = cb == 0 ? first
                                 : (n <= 64 ? __builtin_amdgcn_readlane(sel_mine, cb - 1)
                                            : sel_row[cb - 1]);
        return origin_of(beta) + (uint32_t)(sub_tile_first(g, ct) * (D * 2));
    };

    io.gather(k_rsrc, origin_of_pair(0), tiles_s[0][0]);
    io.gather(v_rsrc, origin_of_pair(0), tiles_s[0][1]);

    // this wavefront's 32 query rows: Q and dO as B operands, lse and delta of
    // the lane's query column
    bf16x8 qf[KS], dof[KS];
    int64_t q_tok;
    {
        const int bw_shift = __builtin_ctz((unsigned)g.block_w);
        const int br = i / g.blocks_per_row, bc = i - br * g.blocks_per_row;
        const int64_t tok0 = (int64_t)br * g.block_h * g.grid_w + (int64_t)bc * g.block_w;
        const int t = 32 * wave + l32;
        const int rr = t >> bw_shift, cc = t & (g.block_w - 1);
        q_tok = tok0 + (int64_t)rr * g.grid_w + cc;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qf[ks] = *(const bf16x8*)(q + base + q_tok * D + 16 * ks + 8 * half);
            dof[ks] = *(const bf16x8*)(dout + base + q_tok * D + 16 * ks + 8 * half);
        }
    }
    const float neg_l2 = -lse2[bh_idx * g.n_tokens + q_tok];
    const float c2 = g.scale * kLog2e;
    // dP^T starts from -delta (a lane's query, so one value), which leaves one
    // product per weight for dS^T = P^T (dP^T - delta)
    f32x16 neg_dl;
    {
        const float x = -delta[bh_idx * g.n_tokens + q_tok];
#pragma unroll
        for (int r = 0; r < 16; ++r) neg_dl[r] = x;
    }

    f32x16 acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = zero_tile();

    if constexpr (D == 64) {
        // Software pipeline over the 32-key halves of the tiles: the
        // exponentials and products that turn S^T, dP^T of one half into dS^T
        // are issued behind the matrix instructions of the next half, two
        // elements per instruction slot, in an order that is written out and
        // pinned (the scheduler would otherwise group them after the matrix
        // instructions, and the two wavefronts of a SIMD do not overlap such
        // phases for each other).  Per tile:
        //   G1  S^T, dP^T of half 0 (8 slots)      | dS^T of the previous half 1
        //   G2  dQ^T += K^T dS^T of the previous half 1 (4 slots),
        //       S^T, dP^T of half 1 (8 slots)      | dS^T of half 0
        //   G3  dQ^T += K^T dS^T of half 0 (4 slots)
        // Carried between tiles: S^T, dP^T of half 1 and its transposed K
        // fragments.
        f32x16 s1, dp1;
#pragma unroll
        for (int r = 0; r < 16; ++r) { s1[r] = -1.0e30f; dp1[r] = 0.0f; }   // weights 0
        bf16x8 ktf[2][2];                                  // [h][dt]
        {
            const bf16x8 z = __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
            ktf[0][0] = z; ktf[0][1] = z; ktf[1][0] = z; ktf[1][1] = z;
        }
        // dS^T of elements 2k, 2k+1 of a half, packed
        auto ds_pair = [&](const f32x16& sv, const f32x16& dpv, int k) -> uint32_t {
            const float f0 = fmaf(sv[2 * k], c2, neg_l2), f1 = fmaf(sv[2 * k + 1], c2, neg_l2);
            const float e0 = __builtin_amdgcn_exp2f(f0), e1 = __builtin_amdgcn_exp2f(f1);
            return pack_bf16(e0 * dpv[2 * k], e1 * dpv[2 * k + 1]);
        };
        // an empty statement that "uses" a slot's result keeps its producers in
        // the slot; no instruction is emitted for it
        auto pin = [](uint32_t& w) {
            asm volatile("" : "+v"(w));
            __builtin_amdgcn_sched_barrier(0);
        };
        for (int c = 0; c < pairs; ++c) {
            // tile c has landed (own loads, then everyone's), every LDS read of
            // the tile before has returned and everyone is done with the other
            // buffer: refill it with tile c + 1
            wait_gathers_and_reads();
            __syncthreads();
            if (c + 1 < pairs) {
                const uint32_t o = origin_of_pair(c + 1);
                io.gather(k_rsrc, o, tiles_s[(c + 1) & 1][0]);
                io.gather(v_rsrc, o, tiles_s[(c + 1) & 1][1]);
            }
            const unsigned char* kt_lds = tiles_s[c & 1][0];
            const unsigned char* vt_lds = tiles_s[c & 1][1];
            bf16x8 kf[KS], vf[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                kf[ks] = row_frag<D>(kt_lds, 0, ks, l32, half);
                vf[ks] = row_frag<D>(vt_lds, 0, ks, l32, half);
            }
            f32x16 s0 = zero_tile(), dp0 = neg_dl;
            uint32_t w[8];
            __builtin_amdgcn_sched_barrier(0);
            // ---- G1
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (k < 4)
                    s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[k], qf[k], s0, 0, 0, 0);
                else
                    dp0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k - 4], dof[k - 4], dp0, 0, 0,
                                                                  0);
                if (k == 3) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) kf[ks] = row_frag<D>(kt_lds, 32, ks, l32, half);
                }
                if (k == 7) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) vf[ks] = row_frag<D>(vt_lds, 32, ks, l32, half);
                }
                w[k] = ds_pair(s1, dp1, k);
                pin(w[k]);
            }
            bf16x8 dsb[2];
            dsb[0] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
            dsb[1] = __builtin_bit_cast(bf16x8, make_uint4(w[4], w[5], w[6], w[7]));
            // ---- G2
            s1 = zero_tile();
            dp1 = neg_dl;
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                if (k < 4)
                    acc[k & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktf[k >> 1][k & 1],
                                                                         dsb[k >> 1], acc[k & 1],
                                                                         0, 0, 0);
                else if (k < 8)
                    s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[k - 4], qf[k - 4], s1, 0, 0, 0);
                else
                    dp1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[k - 8], dof[k - 8], dp1, 0, 0,
                                                                  0);
                if (k == 3) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int dt = 0; dt < DT; ++dt)
                            ktf[h][dt] = trans_frag<D>(kt_lds, 16 * h, dt, lane);
                }
                if (k >= 2 && k < 10) {
                    w[k - 2] = ds_pair(s0, dp0, k - 2);
                    pin(w[k - 2]);
                } else {
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            dsb[0] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
            dsb[1] = __builtin_bit_cast(bf16x8, make_uint4(w[4], w[5], w[6], w[7]));
            // ---- G3
#pragma unroll
            for (int k = 0; k < 4; ++k)
                acc[k & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktf[k >> 1][k & 1], dsb[k >> 1],
                                                                     acc[k & 1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
                    ktf[h][dt] = trans_frag<D>(kt_lds, 32 + 16 * h, dt, lane);
        }
        // the last half 1
        {
            uint32_t w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = ds_pair(s1, dp1, k);
            bf16x8 dsb[2];
            dsb[0] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
            dsb[1] = __builtin_bit_cast(bf16x8, make_uint4(w[4], w[5], w[6], w[7]));
#pragma unroll
            for (int k = 0; k < 4; ++k)
                acc[k & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktf[k >> 1][k & 1], dsb[k >> 1],
                                                                     acc[k & 1], 0, 0, 0);
        }
    } else {
        // Head dim 128.  Per tile of 64 keys, S0 and dP0 of its first half, then S1, dP1,
        // dQ^T += K^T dS^T of half 0 and of half 1, eight matrix instructions each; behind
        // dP0 and dP1 go the exponentials of their half, behind S1 and the first dQ the
        // products.  Fragments are read W instructions ahead.  Against fragments read right
        // before their use and all vector work between the phases (35 % of the wavefronts'
        // cycles were waits): 1.5 degrees, batch 4, 16 heads 2.19 -> 2.03 ms.
        constexpr int ROW = 256, TILE = IO::TILE_BYTES, W = 8;
        uint32_t row_at[4], tr_at[2];
        {
            const uint32_t t0 = lds_address(tiles_s);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                row_at[ks] = t0 + (uint32_t)(l32 * ROW + swz(l32, 2 * ks + half) * 16);
            const int s16 = lane & 15, gq = lane >> 4, r = 4 * (gq >> 1) + (s16 >> 2);
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) {
                const int col = 16 * (gq & 1) + 4 * (s16 & 3) + 32 * dt;
                tr_at[dt] = t0 + (uint32_t)(r * ROW + swz(r, col >> 3) * 16 + (col & 7) * 2);
            }
        }
        // fragment `i` of a tile: K rows, V rows of half 0 (8 each), the same of half 1,
        // K transposed of half 0, of half 1
        auto read_frag = [&](int i) -> bf16x8 {
            const int u = i & 7;
            if (i < 32)
                return lds_read<bf16x8>(row_at[u & 3], ((i >> 3) & 1) * TILE + (i >> 4) * 32 * ROW +
                                                           (u >> 2) * 128);
            const int dt = u & 3, row0 = (i >= 40 ? 32 : 0) + 16 * (u >> 2);
            bf16x4 part[2];
#pragma unroll
            for (int rd = 0; rd < 2; ++rd)
                part[rd] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    (__attribute__((address_space(3))) bf16x4*)(uintptr_t)(
                        tr_at[dt & 1] + (uint32_t)((row0 + 8 * rd) * ROW + (dt >> 1) * 128)));
            return __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
        };
        uint32_t o_next = pairs > 1 ? origin_of_pair(1) : 0u;
        for (int c = 0; c < pairs; ++c) {
            // tile c has landed (own loads, then everyone's) and everyone is done
            // with the other buffer: refill it with tile c + 1
            wait_gathers();
            __syncthreads();
            if (c + 1 < pairs) {
                io.gather(k_rsrc, o_next, tiles_s[(c + 1) & 1][0]);
                io.gather(v_rsrc, o_next, tiles_s[(c + 1) & 1][1]);
            }
            bf16x8 f[W];
            f32x16 s[2], dp[2];
            uint32_t w[2][8];
            float fm[2][2];
#pragma unroll
            for (int i = 0; i < W; ++i) f[i] = read_frag(i);
            s[0] = zero_tile();
            s[1] = zero_tile();
            __builtin_amdgcn_sched_barrier(0);
            auto group = [&](auto g_tag) {
            constexpr int G = decltype(g_tag)::value, hh = (G >> 1) & 1;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int t = 8 * G + u;
                if (G < 4 && (G & 1) == 0)
                    s[hh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[t % W], qf[u], s[hh], 0, 0, 0);
                else if (G < 4)
                    dp[hh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        f[t % W], dof[u], u == 0 ? neg_dl : dp[hh], 0, 0, 0);
                else {
                    const uint32_t(&x)[8] = w[G & 1];
                    const int h = u >> 2;
                    acc[u & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        f[t % W],
                        __builtin_bit_cast(bf16x8, make_uint4(x[4 * h], x[4 * h + 1], x[4 * h + 2],
                                                              x[4 * h + 3])),
                        acc[u & 3], 0, 0, 0);
                }
                if (t + W < 48) f[t % W] = read_frag(t + W);
                // two weights per slot: fma in slot 9 + 16 hh + e/2, the exponentials a slot
                // later, products and packs eight slots after that
                {
                    const int x = t >= 25 ? 1 : 0, e = 2 * (t - 9 - 16 * x);
                    if (e >= 2 && e < 18) {
                        s[x][e - 2] = __builtin_amdgcn_exp2f(fm[t & 1][0]);
                        s[x][e - 1] = __builtin_amdgcn_exp2f(fm[t & 1][1]);
                    }
                    if (e >= 0 && e < 16) {
                        fm[(t + 1) & 1][0] = fmaf(s[x][e], c2, neg_l2);
                        fm[(t + 1) & 1][1] = fmaf(s[x][e + 1], c2, neg_l2);
                        asm volatile("" : "+v"(fm[(t + 1) & 1][0]), "+v"(fm[(t + 1) & 1][1]));
                    }
                }
                {
                    const int x = t >= 34 ? 1 : 0, e = 2 * (t - 18 - 16 * x);
                    if (e >= 0 && e < 16) {
                        w[x][e >> 1] = pack_bf16(s[x][e] * dp[x][e], s[x][e + 1] * dp[x][e + 1]);
                        asm volatile("" : "+v"(w[x][e >> 1]));
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            };
            group(std::integral_constant<int, 0>{});
            group(std::integral_constant<int, 1>{});
            group(std::integral_constant<int, 2>{});
            group(std::integral_constant<int, 3>{});
            group(std::integral_constant<int, 4>{});
            group(std::integral_constant<int, 5>{});
            o_next = c + 2 < pairs ? origin_of_pair(c + 2) : 0u;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) row_at[ks] ^= 2u * TILE;
            tr_at[0] ^= 2u * TILE; tr_at[1] ^= 2u * TILE;
        }
    }

    const float inv_b = 1.0f / (float)g.block_tokens;
    const float* extra = g.add_dq ? g.add_dq + (bh_idx * g.n_blocks + i) * D : nullptr;
    __syncthreads();                                  // the tiles are used up
    unsigned char* const lds = &tiles_s[0][0][0] + wave * 4096;
    uint16_t* const block = dq + base + (origin_of(i) >> 1);
    if (extra) add_rows<D>(block, g, 32 * wave, acc, g.scale, extra, inv_b, lds, lane);
    else store_rows<D>(block, g, 32 * wave, acc, g.scale, lds, lane);
}

// ---------------------------------------------------------------------------
// dK / dV
// ---------------------------------------------------------------------------
// The query blocks connected to key block j, for the query heads of the group that
// share it: heads in ascending order, blocks in ascending order within each, which
// fixes the summation order.  An entry is the first token of the block with the head
// inside the group, counted from head_base, above it (a slice has less than 2^24
// tokens: 32-bit byte offsets).  One wavefront reads 64 words of the reverse map at a
// time, one per lane, and takes as many of them, in order, as the list has room for;
// what is left goes into the next list.
constexpr int kListCap = 1024;
struct ConnectedList {
    uint32_t entry[kListCap];
    int count, more, head_base;
};
__device__ __forceinline__ int fill_list(ConnectedList& list, const Geom& g,
                                         const uint32_t* __restrict__ conn, int64_t bh_first, int j,
                                         int next_word, int lane)
{
    const int m = g.n_blocks, words = (m + 31) >> 5, all_words = g.kv_group * words;
    const int head_base = next_word / words;
    int count = 0;
    bool full = false;
    while (next_word < all_words && !full) {
        const int w = next_word + lane;
        const int head = w / words, wi = w - head * words;
        uint32_t bits = w < all_words ? conn[((bh_first + head) * words + wi) * m + j] : 0u;
        const int mine = __builtin_popcount(bits);
        int upto = mine;                              // inclusive prefix sum over the lanes
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(upto, off);
            upto += lane >= off ? t : 0;
        }
        const uint64_t fits = __builtin_amdgcn_ballot_w64(
            w < all_words && count + upto <= kListCap && head - head_base < 256);
        const int taken = __builtin_popcountll(fits);         // a prefix of the lanes
        if (lane >= taken) bits = 0u;
        int at = count + upto - mine;
        while (bits) {
            const int i = 32 * wi + __builtin_ctz(bits);
            bits &= bits - 1;
            const int br = i / g.blocks_per_row, bc = i - br * g.blocks_per_row;
            list.entry[at++] = (uint32_t)(br * g.block_h * g.grid_w + bc * g.block_w) |
                               (uint32_t)(head - head_base) << 24;
        }
        if (taken > 0) count += __builtin_amdgcn_readlane(upto, taken - 1);
        next_word += taken;
        full = taken < 64;
    }
    if (lane == 0) {
        list.count = count;
        list.more = next_word < all_words ? 1 : 0;
        list.head_base = head_base;
    }
    return next_word;
}

// Launches of few key blocks wait for the longest list (on smooth fields 4 to 7 times the
// mean) while SIMDs are idle.  There SPLIT groups of NW wavefronts own the same key rows
// and take the tiles in turn, with tiles of their own; a block of more than 32 NW rows is
// shared by several workgroups.  add_groups then adds what groups 1 .. have to group 0,
// lane by lane, in the order of the groups, through the tiles' memory (wavefront w of
// group 0 reads only region w, so that it may go on to use it).  All wavefronts call it;
// false: not group 0.
template <int SPLIT, int NW, int COUNT>
__device__ __forceinline__ bool add_groups(unsigned char* lds, int group, int wave, int lane,
                                           f32x16 (&acc)[COUNT])
{
    float* const region = (float*)lds + wave * (SPLIT - 1) * COUNT * 16 * 64 + lane;
    __syncthreads();                                  // the tiles (the last values) are used up
    if (group > 0) {
#pragma unroll
        for (int c = 0; c < COUNT; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                region[(((group - 1) * COUNT + c) * 16 + r) * 64] = acc[c][r];
    }
    __syncthreads();
    if (group > 0) return false;
    for (int from = 0; from < SPLIT - 1; ++from)
#pragma unroll
        for (int c = 0; c < COUNT; ++c) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[c][r] += region[((from * COUNT + c) * 16 + r) * 64];
            __builtin_amdgcn_sched_barrier(0);        // (registers: 16 values at a time)
        }
    lane_exchange();
    return true;
}

// dK and dV in one pass at head dim 64.  What bounds the unpipelined form (fragments
// read right before the matrix instructions, weights between them) is waiting: 44 % of
// the wavefronts' cycles, matrix pipe busy 40 %, and a launch of 16 scan rounds per
// group of 4 heads each of which fills and drains the tile pipeline.  Here
//   * one list holds the connected blocks of the whole group (up to kListCap), its
//     entries are looked up a tile ahead and need no division;
//   * fragments are read W matrix instructions before the one that uses them, in the
//     order of their use: 32 registers that hide the LDS latency at any point;
//   * a tile is two halves of 32 queries: S and dP of half 0, then S and dP of half 1
//     with the weights of half 0 behind them, then dV and dK of half 0 with the weights
//     of half 1, then dV and dK of half 1.  Behind an instruction go the exponentials of
//     two weights, the fma of the next two and the products and packs of the two before,
//     so that nothing waits for the instruction in front of it; the order is written out
//     and pinned.
// 1.5 degree grid, 16 heads on 4, batch 12: 3.83 -> 3.23 ms, its training pass 8.99 -> 8.29 (cycles -23 %: the chip is
// power-limited here and the clock gives part of it back, 1.80 -> 1.62 GHz).
template <int NW, int SUBS, int SPLIT>
__device__ __forceinline__ void dkdv_d64_body(const uint16_t* __restrict__ q,
                                              const uint16_t* __restrict__ k,
                                              const uint16_t* __restrict__ v,
                                              const uint16_t* __restrict__ dout,
                                              const float* __restrict__ lse2,
                                              const float* __restrict__ delta,
                                              const uint32_t* __restrict__ conn,
                                              const int32_t* __restrict__ order,
                                              uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                              const Geom& g, uint32_t n_units)
{
    constexpr int D = 64, KS = 4, ROW = 128, TILE = 64 * ROW, CHUNKS = 2 * SUBS / NW;
    using IO = TileIO<D, NW>;
    // [buffer][Q tile, dO tile]; the buffers alternate by bit 14 of the address
    __shared__ __attribute__((aligned(32768))) unsigned char tiles_s[SPLIT][2][2][TILE];
    __shared__ __attribute__((aligned(1024))) float rows_s[SPLIT][2][2][64];  // [buffer][lse2, delta]
    __shared__ ConnectedList list;

    const int lane = threadIdx.x & 63;
    const int wg_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = SPLIT == 1 ? 0 : wg_wave / NW, wave = wg_wave - group * NW;
    const int l32 = lane & 31, half = lane >> 5;
    const int m = g.n_blocks;

    // workgroup -> (key/value slice, key block); the query slices that share the
    // key/value slice are consecutive
    uint32_t unit, r_unit;
    map_key_block(g, blockIdx.x, CHUNKS, n_units, unit, r_unit);
    const int place = (int)r_unit / CHUNKS, row0 = 32 * (NW * ((int)r_unit % CHUNKS) + wave);
    const int j = order ? order[(int64_t)unit * m + place] : place;
    const int64_t base = (int64_t)unit * g.n_tokens * D;
    int64_t bh_first;
    {
        const uint32_t kv_heads = (uint32_t)(g.heads / g.kv_group);
        const uint32_t e = unit / kv_heads, a = unit - e * kv_heads;
        bh_first = (int64_t)e * g.heads + (int64_t)a * g.kv_group;
    }
    const uint32_t slice_bytes = (uint32_t)(g.n_tokens * D * 2), row_bytes = (uint32_t)(g.n_tokens * 4);

    IO io;
    io.init(g, lane, wave);

    // this wavefront's 32 key rows: K and -V as B operands
    bf16x8 kfb[KS], vfb[KS];
    int64_t k_tok;
    {
        const int bw_shift = __builtin_ctz((unsigned)g.block_w);
        const int br = j / g.blocks_per_row, bc = j - br * g.blocks_per_row;
        const int64_t tok0 = (int64_t)br * g.block_h * g.grid_w + (int64_t)bc * g.block_w;
        const int t = row0 + l32;
        const int rr = t >> bw_shift, cc = t & (g.block_w - 1);
        k_tok = tok0 + (int64_t)rr * g.grid_w + cc;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            kfb[ks] = *(const bf16x8*)(k + base + k_tok * D + 16 * ks + 8 * half);
            vfb[ks] = negated(*(const bf16x8*)(v + base + k_tok * D + 16 * ks + 8 * half));
        }
    }
    const float c2 = g.scale * kLog2e;

    f32x16 acck[2], accv[2];
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) acck[dt] = accv[dt] = zero_tile();

    // addresses of this lane's fragments (row_frag, trans_frag) in the buffer that is
    // read next; everything else is a constant
    uint32_t row_at[KS], tr_at[2], val_at;
    {
        const uint32_t t0 = lds_address(tiles_s[0]) + (uint32_t)group * (4u * TILE);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            row_at[ks] = t0 + (uint32_t)(l32 * ROW + swz(l32, 2 * ks + half) * 16);
        const int s16 = lane & 15, gq = lane >> 4, r = 4 * (gq >> 1) + (s16 >> 2);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            const int col = 16 * (gq & 1) + 4 * (s16 & 3) + 32 * dt;
            tr_at[dt] = t0 + (uint32_t)(r * ROW + swz(r, col >> 3) * 16 + (col & 7) * 2);
        }
        val_at = lds_address(rows_s[0]) + 1024u * (uint32_t)group + 16u * (uint32_t)half;
    }
    // fragment `i` of a tile in the order in which the matrix instructions take them:
    //   0- 7  Q rows, dO rows of queries 0..31 (S, dP)     8-15  the same of 32..63
    //  16-23  dO, Q transposed of queries 0..31 (dV, dK)  24-31  the same of 32..63
    auto read_frag = [&](int i) -> bf16x8 {
        const int u = i & 3;
        if (i < 16) {
            const int qt = i >> 3, is_g = (i >> 2) & 1;
            return lds_read<bf16x8>(row_at[u], is_g * TILE + qt * 32 * ROW);
        }
        const int qt = (i - 16) >> 3, is_g = 1 - ((i >> 2) & 1), h = u >> 1, dt = u & 1;
        bf16x4 part[2];
#pragma unroll
        for (int rd = 0; rd < 2; ++rd)
            part[rd] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                (__attribute__((address_space(3))) bf16x4*)(uintptr_t)(
                    tr_at[dt] + (uint32_t)(is_g * TILE + (32 * qt + 16 * h + 8 * rd) * ROW)));
        return __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
    };

    int next_word = 0;                                // the first wavefront only
    for (;;) {
        __syncthreads();                              // the previous list is used up
        if (wg_wave == 0) next_word = fill_list(list, g, conn, bh_first, j, next_word, lane);
        __syncthreads();
        const int items = __builtin_amdgcn_readfirstlane(list.count) * SUBS;
        const bool more = __builtin_amdgcn_readfirstlane(list.more) != 0;
        const int64_t bh0 = bh_first + __builtin_amdgcn_readfirstlane(list.head_base);

        auto entry_of = [&](int item) -> uint32_t { return list.entry[min(item, items - 1) / SUBS]; };
        auto issue_item = [&](int item, uint32_t entry, int buf) {
            const uint64_t bh = (uint64_t)(bh0 + (entry >> 24));
            const uint32_t tok = (entry & 0xffffffu) + (uint32_t)sub_tile_first(g, item % SUBS);
            const i32x4 q_rsrc = buffer_desc((const char*)q + bh * slice_bytes, slice_bytes);
            const i32x4 g_rsrc = buffer_desc((const char*)dout + bh * slice_bytes, slice_bytes);
            io.gather(q_rsrc, tok * ROW, tiles_s[group][buf][0]);
            io.gather(g_rsrc, tok * ROW, tiles_s[group][buf][1]);
            if (wave == 0)
                io.gather_f32(buffer_desc((const char*)lse2 + bh * row_bytes, row_bytes), tok,
                              rows_s[group][buf][0]);
            if (wave == NW - 1)
                io.gather_f32(buffer_desc((const char*)delta + bh * row_bytes, row_bytes), tok,
                              rows_s[group][buf][1]);
        };
        if (items > 0) {
            uint32_t entry = __builtin_amdgcn_readfirstlane(entry_of(group));
            if (SPLIT == 1 || group < items) issue_item(group, entry, 0);
            entry = __builtin_amdgcn_readfirstlane(entry_of(group + SPLIT));
            // tile 0 of a list lies in buffer 0
            const uint32_t flip = row_at[0] & 16384u;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) row_at[ks] -= flip;
            tr_at[0] -= flip; tr_at[1] -= flip;
            val_at -= flip >> 5;
            for (int it0 = 0; it0 < items; it0 += SPLIT) {
                // item `it` has landed and everyone is done with the other buffers
                wait_gathers();
                __syncthreads();
                const int it = it0 + group;
                if (SPLIT > 1 && it >= items) break;          // the last round
                if (it + SPLIT < items) issue_item(it + SPLIT, entry, (it0 / SPLIT + 1) & 1);
                const uint32_t entry_v = entry_of(it + 2 * SPLIT);

                constexpr int W = 8;                  // fragments read ahead
                bf16x8 f[W];
                f32x16 s[2], dp[2];
                f32x4 l4[4];
                uint32_t pw[2][8], dw[2][8];
                float fm[2][2], ex[2][2];
                // delta - dP: the accumulator starts from delta, one value per row, as
                // it lies in LDS (element r is query row 8 (r/4) + 4 half + r%4)
                auto read_delta = [&](int qt) {
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const f32x4 d4 = lds_read<f32x4>(val_at, 256 + 128 * qt + 32 * r4);
#pragma unroll
                        for (int r = 0; r < 4; ++r) dp[qt][4 * r4 + r] = d4[r];
                    }
                };
#pragma unroll
                for (int i = 0; i < 4; ++i) f[i] = read_frag(i);
                read_delta(0);
#pragma unroll
                for (int i = 4; i < W; ++i) f[i] = read_frag(i);
                s[0] = zero_tile();
                s[1] = zero_tile();
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    const int u = i & 3;
                    const bf16x8 x = f[i % W];
                    if (i < 16) {
                        const int qt = i >> 3;
                        if ((i & 4) == 0)
                            s[qt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, kfb[u], s[qt], 0, 0, 0);
                        else
                            dp[qt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, vfb[u], dp[qt], 0, 0, 0);
                    } else {
                        const int qt = (i - 16) >> 3, h = u >> 1, dt = u & 1;
                        const uint32_t(&w)[8] = (i & 4) == 0 ? pw[qt] : dw[qt];
                        const bf16x8 b = __builtin_bit_cast(
                            bf16x8, make_uint4(w[4 * h], w[4 * h + 1], w[4 * h + 2], w[4 * h + 3]));
                        if ((i & 4) == 0)
                            accv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, b, accv[dt], 0, 0, 0);
                        else
                            acck[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, b, acck[dt], 0, 0, 0);
                    }
                    if (i + W < 32) f[i % W] = read_frag(i + W);
                    // lse of the queries whose weights come next, delta of the second half
                    if (i >= 3 && i < 7) l4[i - 3] = lds_read<f32x4>(val_at, 32 * (i - 3));
                    if (i == 7) read_delta(1);
                    if (i >= 10 && i < 18 && (i & 1) == 0)
                        l4[(i - 10) >> 1] = lds_read<f32x4>(val_at, 128 + 32 * ((i - 10) >> 1));
                    // weights of half qt behind the instructions 8 + 8 qt ..: per slot the
                    // exponentials of two elements, the fma of the next two and the products
                    // and packs of the two before
                    if (i >= 7 && i < 23) {
                        const int qt = (i - 7) >> 3, e = 2 * ((i - 7) & 7);
                        fm[(i + 1) & 1][0] = fmaf(s[qt][e], c2, -l4[e >> 2][e & 3]);
                        fm[(i + 1) & 1][1] = fmaf(s[qt][e + 1], c2, -l4[e >> 2][(e & 3) + 1]);
                        asm volatile("" : "+v"(fm[(i + 1) & 1][0]), "+v"(fm[(i + 1) & 1][1]));
                    }
                    if (i >= 8 && i < 24) {
                        ex[i & 1][0] = __builtin_amdgcn_exp2f(fm[i & 1][0]);
                        ex[i & 1][1] = __builtin_amdgcn_exp2f(fm[i & 1][1]);
                        asm volatile("" : "+v"(ex[i & 1][0]), "+v"(ex[i & 1][1]));
                    }
                    if (i >= 9 && i < 25) {
                        const int qt = (i - 9) >> 3, e = 2 * ((i - 9) & 7), o = (i - 1) & 1;
                        pw[qt][e >> 1] = pack_bf16(ex[o][0], ex[o][1]);
                        dw[qt][e >> 1] = pack_bf16(ex[o][0] * dp[qt][e], ex[o][1] * dp[qt][e + 1]);
                        asm volatile("" : "+v"(pw[qt][e >> 1]), "+v"(dw[qt][e >> 1]));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                entry = __builtin_amdgcn_readfirstlane(entry_v);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) row_at[ks] ^= 16384u;
                tr_at[0] ^= 16384u; tr_at[1] ^= 16384u;
                val_at ^= 512u;
            }
        }
        if (!more) break;
    }

    const float inv_b = 1.0f / (float)g.block_tokens;
    const int64_t pooled_row = ((int64_t)unit * m + j) * D;
    const float* extra_k = g.add_dk ? g.add_dk + pooled_row : nullptr;
    const float* extra_v = g.add_dv ? g.add_dv + pooled_row : nullptr;
    unsigned char* lds = &tiles_s[0][0][0][0];
    if constexpr (SPLIT > 1) {
        static_assert(NW * (SPLIT - 1) * 2 * 4096 <= (int)sizeof(tiles_s), "fits the tiles");
        const bool first = add_groups<SPLIT, NW>(lds, group, wave, lane, acck);
        if (!add_groups<SPLIT, NW>(lds, group, wave, lane, accv) || !first) return;
        lds += wave * (SPLIT - 1) * 2 * 4096;
    } else {
        __syncthreads();                              // the tiles are used up
        lds += wave * 4096;
    }
    const int br = j / g.blocks_per_row, bc = j - br * g.blocks_per_row;
    const int64_t block =
        base + ((int64_t)br * g.block_h * g.grid_w + (int64_t)bc * g.block_w) * D;
    if (extra_k) add_rows<D>(dk + block, g, row0, acck, -g.scale, extra_k, inv_b, lds, lane);
    else store_rows<D>(dk + block, g, row0, acck, -g.scale, lds, lane);
    if (extra_v) add_rows<D>(dv + block, g, row0, accv, 1.0f, extra_v, inv_b, lds, lane);
    else store_rows<D>(dv + block, g, row0, accv, 1.0f, lds, lane);
}

// dK and dV in one pass at head dim 128.  Both accumulators take 128 of the 256 registers
// that two wavefronts per SIMD leave, K 32; V lies in LDS (negated, each wavefront its own
// 32 rows) and its fragments are read with those of dO.  Tiles of 32 queries, so that two
// workgroups (blocks of 256: one) fit a CU beside it.  Fragments are read W of them ahead
// in the order of their use; the exponentials go behind the dP instructions, the products
// behind those of dV.  Against a pass each for dV and dK, which compute S twice, gather
// every tile twice and wait 40 % of the time for fragments: 1.5 degrees, batch 4, 16 heads
// 1.85 + 2.38 -> 3.23 ms, training pass 8.65 -> 7.56; the same bits.
template <int NW, int SUBS, int SPLIT>
__device__ __forceinline__ void dkdv_d128_body(const uint16_t* __restrict__ q,
                                               const uint16_t* __restrict__ k,
                                               const uint16_t* __restrict__ v,
                                               const uint16_t* __restrict__ dout,
                                               const float* __restrict__ lse2,
                                               const float* __restrict__ delta,
                                               const uint32_t* __restrict__ conn,
                                               const int32_t* __restrict__ order,
                                               uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                               const Geom& g, uint32_t n_units)
{
    constexpr int D = 128, KS = 8, ROW = 256, TILE = 32 * ROW, MINE = 8 / NW, CHUNKS = SUBS / NW;
    // [buffer][Q tile, dO tile]; the buffers alternate by bit 14 of the address
    __shared__ __attribute__((aligned(32768))) unsigned char tiles_s[SPLIT][2][2][TILE];
    __shared__ __attribute__((aligned(1024))) float rows_s[SPLIT][2][2][64];  // [buffer][lse2, delta]
    __shared__ __attribute__((aligned(1024))) unsigned char v_s[NW][TILE];
    __shared__ ConnectedList list;

    const int lane = threadIdx.x & 63;
    const int wg_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = SPLIT == 1 ? 0 : wg_wave / NW, wave = wg_wave - group * NW;
    const int l32 = lane & 31, half = lane >> 5;
    const int m = g.n_blocks;

    // workgroup -> (key/value slice, key block), see dkdv_d64_body
    uint32_t unit, r_unit;
    map_key_block(g, blockIdx.x, CHUNKS, n_units, unit, r_unit);
    const int place = (int)r_unit / CHUNKS, row0 = 32 * (NW * ((int)r_unit % CHUNKS) + wave);
    const int j = order ? order[(int64_t)unit * m + place] : place;
    const int64_t base = (int64_t)unit * g.n_tokens * D;
    int64_t bh_first;
    {
        const uint32_t kv_heads = (uint32_t)(g.heads / g.kv_group);
        const uint32_t e = unit / kv_heads, a = unit - e * kv_heads;
        bh_first = (int64_t)e * g.heads + (int64_t)a * g.kv_group;
    }
    const uint32_t slice_bytes = (uint32_t)(g.n_tokens * D * 2), row_bytes = (uint32_t)(g.n_tokens * 4);

    // gathers: slab wave + NW jj holds tile rows 4 slab .. + 3
    uint32_t voff[MINE];
#pragma unroll
    for (int jj = 0; jj < MINE; ++jj) {
        const int t = 4 * (wave + NW * jj) + (lane >> 4);
        voff[jj] = (uint32_t)(sub_tile_pos(g, t) * ROW + swz(t, lane & 15) * 16);
    }
    const uint32_t tok_off = (uint32_t)(sub_tile_pos(g, l32) * 4);

    // this wavefront's 32 key rows: K as B operand, -V to LDS
    bf16x8 kfb[KS];
    int64_t k_tok;
    {
        const int bw_shift = __builtin_ctz((unsigned)g.block_w);
        const int br = j / g.blocks_per_row, bc = j - br * g.blocks_per_row;
        const int64_t tok0 = (int64_t)br * g.block_h * g.grid_w + (int64_t)bc * g.block_w;
        const int t = row0 + l32;
        const int rr = t >> bw_shift, cc = t & (g.block_w - 1);
        k_tok = tok0 + (int64_t)rr * g.grid_w + cc;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            kfb[ks] = *(const bf16x8*)(k + base + k_tok * D + 16 * ks + 8 * half);
            if (SPLIT > 1 && group > 0) continue;     // V is the same for all groups
            *(bf16x8*)(v_s[wave] + l32 * ROW + swz(l32, 2 * ks + half) * 16) =
                negated(*(const bf16x8*)(v + base + k_tok * D + 16 * ks + 8 * half));
        }
    }
    const float c2 = g.scale * kLog2e;

    f32x16 acck[4], accv[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) acck[dt] = accv[dt] = zero_tile();

    // addresses of this lane's fragments (row_frag, trans_frag) in the buffer that is
    // read next, and of its V rows; everything else is a constant
    uint32_t row_at[4], v_at[4], tr_at[2], val_at;
    {
        const uint32_t t0 = lds_address(tiles_s[0]) + (uint32_t)group * (4u * TILE), v0 = lds_address(v_s[0]) + (uint32_t)wave * TILE;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const uint32_t at = (uint32_t)(l32 * ROW + swz(l32, 2 * ks + half) * 16);
            row_at[ks] = t0 + at;
            v_at[ks] = v0 + at;
        }
        const int s16 = lane & 15, gq = lane >> 4, r = 4 * (gq >> 1) + (s16 >> 2);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            const int col = 16 * (gq & 1) + 4 * (s16 & 3) + 32 * dt;
            tr_at[dt] = t0 + (uint32_t)(r * ROW + swz(r, col >> 3) * 16 + (col & 7) * 2);
        }
        val_at = lds_address(rows_s[0]) + 1024u * (uint32_t)group + 16u * (uint32_t)half;
    }
    // fragment `i` of a tile in the order in which the matrix instructions take them:
    // 0-7 Q rows (S), 8-23 dO rows and V in turn (dP), 24-31 dO transposed (dV),
    // 32-39 Q transposed (dK)
    auto read_frag = [&](int i) -> bf16x8 {
        if (i < 24) {
            const int ks = i < 8 ? i : (i - 8) >> 1, imm = (ks >> 2) * 128;
            if (i >= 8 && (i & 1)) return lds_read<bf16x8>(v_at[ks & 3], imm);
            return lds_read<bf16x8>(row_at[ks & 3], imm + (i >= 8 ? TILE : 0));
        }
        const int is_g = i < 32, h = (i >> 2) & 1, dt = i & 3;
        bf16x4 part[2];
#pragma unroll
        for (int rd = 0; rd < 2; ++rd)
            part[rd] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                (__attribute__((address_space(3))) bf16x4*)(uintptr_t)(
                    tr_at[dt & 1] +
                    (uint32_t)(is_g * TILE + (16 * h + 8 * rd) * ROW + (dt >> 1) * 128)));
        return __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
    };

    int next_word = 0;                                // the first wavefront only
    for (;;) {
        __syncthreads();                              // the previous list is used up
        if (wg_wave == 0) next_word = fill_list(list, g, conn, bh_first, j, next_word, lane);
        __syncthreads();
        const int items = __builtin_amdgcn_readfirstlane(list.count) * SUBS;
        const bool more = __builtin_amdgcn_readfirstlane(list.more) != 0;
        const int64_t bh0 = bh_first + __builtin_amdgcn_readfirstlane(list.head_base);

        auto entry_of = [&](int item) -> uint32_t { return list.entry[min(item, items - 1) / SUBS]; };
        auto issue_item = [&](int item, uint32_t entry, int buf) {
            const uint64_t bh = (uint64_t)(bh0 + (entry >> 24));
            const int ct = item % SUBS;
            const uint32_t tok = (entry & 0xffffffu) + (uint32_t)sub_tile_first(g, ct >> 1) +
                                 (uint32_t)((ct & 1) * sub_tile_pos(g, 32));
            const i32x4 q_rsrc = buffer_desc((const char*)q + bh * slice_bytes, slice_bytes);
            const i32x4 g_rsrc = buffer_desc((const char*)dout + bh * slice_bytes, slice_bytes);
            const uint32_t q_dst = lds_address(tiles_s[group][buf][0]), g_dst = lds_address(tiles_s[group][buf][1]);
#pragma unroll
            for (int jj = 0; jj < MINE; ++jj) {
                load_lds_16(q_rsrc, voff[jj], tok * ROW, q_dst + (uint32_t)(wave + NW * jj) * 1024u);
                load_lds_16(g_rsrc, voff[jj], tok * ROW, g_dst + (uint32_t)(wave + NW * jj) * 1024u);
            }
            if (wave == 0)
                load_lds_4(buffer_desc((const char*)lse2 + bh * row_bytes, row_bytes), tok_off,
                           tok * 4u, lds_address(rows_s[group][buf][0]));
            if (wave == NW - 1)
                load_lds_4(buffer_desc((const char*)delta + bh * row_bytes, row_bytes), tok_off,
                           tok * 4u, lds_address(rows_s[group][buf][1]));
        };
        if (items > 0) {
            uint32_t entry = __builtin_amdgcn_readfirstlane(entry_of(group));
            if (SPLIT == 1 || group < items) issue_item(group, entry, 0);
            entry = __builtin_amdgcn_readfirstlane(entry_of(group + SPLIT));
            // tile 0 of a list lies in buffer 0
            const uint32_t flip = row_at[0] & 16384u;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) row_at[ks] -= flip;
            tr_at[0] -= flip; tr_at[1] -= flip;
            val_at -= flip >> 5;
            for (int it0 = 0; it0 < items; it0 += SPLIT) {
                // item `it` has landed and everyone is done with the other buffers
                wait_gathers();
                __syncthreads();
                const int it = it0 + group;
                if (SPLIT > 1 && it >= items) break;          // the last round
                if (it + SPLIT < items) issue_item(it + SPLIT, entry, (it0 / SPLIT + 1) & 1);
                const uint32_t entry_v = entry_of(it + 2 * SPLIT);

                constexpr int W = 6;                  // fragments read ahead
                bf16x8 f[W];
                f32x16 s = zero_tile(), dp;
                f32x4 l4[2];
                uint32_t pw[8], dw[8];
                float fm[2][2];
#pragma unroll
                for (int i = 0; i < W; ++i) f[i] = read_frag(i);
                __builtin_amdgcn_sched_barrier(0);
                // the fragment that a slot's instruction has taken makes room for the one W
                // further on
                auto ask = [&](int i) {
                    if (i + W < 40) f[i % W] = read_frag(i + W);
                };
                auto operand = [](const uint32_t(&w)[8], int h) {
                    return __builtin_bit_cast(
                        bf16x8, make_uint4(w[4 * h], w[4 * h + 1], w[4 * h + 2], w[4 * h + 3]));
                };
#pragma unroll
                for (int t = 0; t < 32; ++t) {
                    const int i = t & 7, h = i >> 2, dt = i & 3;
                    if (t < 8) {
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % W], kfb[i], s, 0, 0, 0);
                        ask(i);
                    } else if (t < 16) {
                        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            f[(8 + 2 * i) % W], f[(9 + 2 * i) % W], dp, 0, 0, 0);
                        ask(8 + 2 * i);
                        ask(9 + 2 * i);
                    } else if (t < 24) {
                        accv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            f[(24 + i) % W], operand(pw, h), accv[dt], 0, 0, 0);
                        ask(24 + i);
                    } else {
                        acck[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            f[(32 + i) % W], operand(dw, h), acck[dt], 0, 0, 0);
                        ask(32 + i);
                    }
                    // delta - dP: the accumulator starts from delta, one value per row, as
                    // it lies in LDS (element r is query row 8 (r/4) + 4 half + r%4)
                    if (t >= 2 && t < 6) {
                        const f32x4 d4 = lds_read<f32x4>(val_at, 256 + 32 * (t - 2));
#pragma unroll
                        for (int r = 0; r < 4; ++r) dp[4 * (t - 2) + r] = d4[r];
                    }
                    if (t == 6 || t == 7) l4[t - 6] = lds_read<f32x4>(val_at, 32 * (t - 6));
                    // two weights: the fma in slot 9 + e/2, the exponentials (and P) a slot
                    // later, the products (-dS; the sign goes into the scale of dK) behind
                    // dV and the first of dK
                    if (t >= 10 && t < 18) {
                        const int e = 2 * (t - 10);
                        s[e] = __builtin_amdgcn_exp2f(fm[t & 1][0]);
                        s[e + 1] = __builtin_amdgcn_exp2f(fm[t & 1][1]);
                        pw[e >> 1] = pack_bf16(s[e], s[e + 1]);
                        asm volatile("" : "+v"(pw[e >> 1]));
                    }
                    if (t >= 9 && t < 17) {
                        const int e = 2 * (t - 9);
                        fm[(t + 1) & 1][0] = fmaf(s[e], c2, -l4[(e >> 2) & 1][e & 3]);
                        fm[(t + 1) & 1][1] = fmaf(s[e + 1], c2, -l4[(e >> 2) & 1][(e & 3) + 1]);
                        asm volatile("" : "+v"(fm[(t + 1) & 1][0]), "+v"(fm[(t + 1) & 1][1]));
                    }
                    if (t == 10 || t == 12) l4[(t - 10) >> 1] = lds_read<f32x4>(val_at, 64 + 16 * (t - 10));
                    if (t >= 18 && t < 26) {
                        const int e = 2 * (t - 18);
                        dw[e >> 1] = pack_bf16(s[e] * dp[e], s[e + 1] * dp[e + 1]);
                        asm volatile("" : "+v"(dw[e >> 1]));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                entry = __builtin_amdgcn_readfirstlane(entry_v);
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) row_at[ks] ^= 16384u;
                tr_at[0] ^= 16384u; tr_at[1] ^= 16384u;
                val_at ^= 512u;
            }
        }
        if (!more) break;
    }

    const float inv_b = 1.0f / (float)g.block_tokens;
    const int64_t pooled_row = ((int64_t)unit * m + j) * D;
    const float* extra_k = g.add_dk ? g.add_dk + pooled_row : nullptr;
    const float* extra_v = g.add_dv ? g.add_dv + pooled_row : nullptr;
    unsigned char* lds = &tiles_s[0][0][0][0];
    if constexpr (SPLIT > 1) {
        static_assert(NW * (SPLIT - 1) * 4 * 4096 <= (int)sizeof(tiles_s), "fits the tiles");
        const bool first = add_groups<SPLIT, NW>(lds, group, wave, lane, acck);
        if (!add_groups<SPLIT, NW>(lds, group, wave, lane, accv) || !first) return;
        lds += wave * (SPLIT - 1) * 4 * 4096;
    } else {
        __syncthreads();                              // the tiles are used up
        lds += wave * 4096;
    }
    const int br = j / g.blocks_per_row, bc = j - br * g.blocks_per_row;
    const int64_t block =
        base + ((int64_t)br * g.block_h * g.grid_w + (int64_t)bc * g.block_w) * D;
    if (extra_k) add_rows<D>(dk + block, g, row0, acck, -g.scale, extra_k, inv_b, lds, lane);
    else store_rows<D>(dk + block, g, row0, acck, -g.scale, lds, lane);
    if (extra_v) add_rows<D>(dv + block, g, row0, accv, 1.0f, extra_v, inv_b, lds, lane);
    else store_rows<D>(dv + block, g, row0, accv, 1.0f, lds, lane);
}

}  // namespace bwdm

// plain kernels per (head dim, wavefronts per workgroup); the bodies are templates
#define BSA_BWD_DQ(D, NW)                                                                         \
    __global__ __launch_bounds__(64 * NW, 2) void bwd_mfma_dq_d##D##_w##NW(                       \
        const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* dout,            \
        const float* lse2, const float* delta, const int32_t* sel_idx, uint16_t* dq, Geom g,      \
        uint32_t n_units)                                                                       \
    {                                                                                             \
        bwdm::dq_body<D, NW>(q, k, v, dout, lse2, delta, sel_idx, dq, g, n_units);             \
    }
BSA_BWD_DQ(64, 2)
BSA_BWD_DQ(64, 4)
BSA_BWD_DQ(64, 8)
BSA_BWD_DQ(128, 4)
BSA_BWD_DQ(128, 8)
// NW wavefronts of 32 rows per workgroup (times the groups), SUBS tiles per query block
#define BSA_BWD_DKDV(NAME, D, NW, SUBS, SPLIT)                                                    \
    __global__ __launch_bounds__(64 * NW * SPLIT, D == 128 && NW * SPLIT == 4 && SPLIT > 1 ? 1 : 2)      \
    void bwd_mfma_dkdv_d##D##_##NAME(                                                             \
        const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* dout,            \
        const float* lse2, const float* delta, const uint32_t* conn, const int32_t* order,        \
        uint16_t* dk, uint16_t* dv, Geom g, uint32_t n_units)                                     \
    {                                                                                             \
        bwdm::dkdv_d##D##_body<NW, SUBS, SPLIT>(q, k, v, dout, lse2, delta, conn, order, dk, dv,  \
                                                g, n_units);                                      \
    }
BSA_BWD_DKDV(w2, 64, 2, 1, 1)
BSA_BWD_DKDV(w4, 64, 4, 2, 1)
BSA_BWD_DKDV(w8, 64, 8, 4, 1)
BSA_BWD_DKDV(w2_split2, 64, 2, 1, 2)
BSA_BWD_DKDV(w4_split2, 64, 2, 2, 2)
BSA_BWD_DKDV(w8_split2, 64, 2, 4, 2)
BSA_BWD_DKDV(w2_split4, 64, 2, 1, 4)
BSA_BWD_DKDV(w4_split4, 64, 2, 2, 4)
BSA_BWD_DKDV(w8_split4, 64, 2, 4, 4)
BSA_BWD_DKDV(w4, 128, 4, 4, 1)
BSA_BWD_DKDV(w8, 128, 8, 8, 1)
BSA_BWD_DKDV(w4_split2, 128, 2, 4, 2)
BSA_BWD_DKDV(w8_split2, 128, 2, 8, 2)
BSA_BWD_DKDV(w8_split2_wide, 128, 4, 8, 2)
#undef BSA_BWD_DQ
#undef BSA_BWD_DKDV

bool bwd_mfma_supported(bool is_bf16, const Geom& g, int D)
{
    // a wavefront per 32 rows of a block of 64, 128 or 256 tokens; 64-token
    // sub-tiles (tile width a power of two: whole tile rows, or 64-token runs of
    // one row); 32-bit buffer offsets inside a slice
    // (head dim 128 with 64-token blocks would leave one wavefront per SIMD)
    const int b = g.block_tokens;
    return is_bf16 && (D == 64 || D == 128) && (b == 64 || b == 128 || b == 256) &&
           !(D == 128 && b == 64) &&
           (g.block_w & (g.block_w - 1)) == 0 && g.n_tokens * D * 2 < ((int64_t)1 << 31);
}

// Wavefronts of 32 rows of a dK/dV workgroup, and groups of them that share its list, by
// the row wavefronts of the launch and the tiles' worth of rows (32) that one walks on
// average.  What bounds a launch of few wavefronts and what a split costs is said at the
// general kernels' rule (bsa_bwd.hip).  Whole backward, us, unsplit | two wavefronts in two
// groups | in four (slices x blocks x tokens, attended blocks; head dim 128, last: four
// wavefronts in two groups):
//   head dim 64:   1 x 24 x 128, 13:   78 | 62 | 58       4 x 96 x 128, 13:   154 | 136 | 129
//                  1 x 448 x 64, 13:   88 | 74 | 70       4 x 448 x 64, 13:   163 | 154 | 175
//                  1 x 448 x 128, 4:   92 | 72 | 77       16 x 96 x 128, 13:  324 | 330 | 376
//                  4 x 96 x 256, 13:  411 | 357 | 377     16 x 96 x 256, 13: 1,185 | 1,161 | 1,247
//   head dim 128:  1 x 96 x 128, 13:  185 | 132 | -       4 x 96 x 128, 13:   249 | 221 | -
//                  16 x 96 x 128, 13: 580 | 690 | -       4 x 96 x 256, 13:   727 | 720 | 655
//                  1 x 448 x 256, 4:  340 | 309 | 277     16 x 96 x 256, 13: 2,256 | 2,480 | 2,234
// (four groups at head dim 128 take 155 KB of LDS beside V; built, they spilled and were no faster
// than two).  Lists of equal length (see there) are
// split while SIMDs are idle.  367 launches of 48 to 12,288 row wavefronts, smooth fields,
// noise, n = 0 and all blocks: 1.18 (head dim 64) and 1.20 times as fast on average; of 200
// others, up to 9,000, five were slower than unsplit by 2 to 9 %.  The terms a + w / c: see there.
struct DkdvSplit {
    int waves, groups;
};
static DkdvSplit dkdv_split(const Geom& g, int D, int64_t BKV)
{
    const int nw = g.block_tokens / 32;
    const int64_t waves = BKV * g.n_blocks * nw, attended = g.n_select + 1 - g.list_only;
    const int64_t pieces = g.kv_group * attended * nw;
    const bool even = g.add_dk || attended == 1 || 2 * attended > g.n_blocks;
    const int64_t few = even ? 2048 / 3 : 2048, more = even ? 1024 : 4096;
    if (D == 64) {
        if (waves <= few && pieces >= 16 + waves / 64) return {2, 4};
        if (waves <= more && pieces >= 8 + waves / 256) return {2, 2};
    } else {
        if (waves <= few && pieces >= 6 + waves / 128) return {2, 2};
        if (nw == 8 && waves <= more && pieces >= 6 + waves / 256) return {4, 2};
    }
    return {nw, 1};
}

hipError_t launch_bwd_mfma(const void* q, const void* k, const void* v, const void* out,
                           const float* lse, const void* dout, const int32_t* sel_idx, void* dq,
                           void* dk, void* dv, float* delta, float* lse2, uint32_t* conn, int32_t* order,
                           const Geom& g, int D, int64_t BH, hipStream_t stream)
{
    const int nw = g.block_tokens / 32;
    const uint32_t sx = (uint32_t)(BH / g.kv_group);           // key/value slices
    const DkdvSplit split = dkdv_split(g, D, sx);
    auto run = [&](auto dq_kernel, auto dkdv_kernel) {
        const bool dkdv_first = order != nullptr;    // `order` may lie where dQ goes
        const int waves = split.waves * split.groups;
        const uint32_t wgs = sx * (unsigned)(g.n_blocks * (nw / split.waves));
        const bool even = even_lists(g);
        if (even || (order && needs_no_order(dkdv_kernel, wgs, waves, 0, short_lists(g, D, false))))
            order = nullptr;
        hipError_t e = launch_bwd_prepare(true, out, dout, lse, delta, lse2, sel_idx, conn, order, g,
                                          D, BH, stream);
        if (e != hipSuccess) return e;
        auto run_dkdv = [&] {
            Geom gk = g;
            gk.deal = key_deal(g.deal, 2 * g.n_tokens * D * 2, order != nullptr, even);
            dkdv_kernel<<<dim3(wgs), dim3(64 * waves), 0, stream>>>(
                (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout,
                lse2, delta, conn, order, (uint16_t*)dk, (uint16_t*)dv, gk, sx);
            return hipGetLastError();
        };
        auto run_dq = [&] {
            dq_kernel<<<dim3((unsigned)(BH * g.n_blocks)), dim3(64 * nw), 0, stream>>>(
                (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout,
                lse2, delta, sel_idx, (uint16_t*)dq, g, sx);
            return hipGetLastError();
        };
        // without the memory for an order dK and dV may lie where k and v are
        e = dkdv_first ? run_dkdv() : run_dq();
        if (e != hipSuccess) return e;
        return dkdv_first ? run_dq() : run_dkdv();
    };
#define BSA_LAUNCH(D_, NW_, FOUR_GROUPS, FOUR_WAVES)                                              \
    if (D == D_ && nw == NW_)                                                                     \
        return run(bwd_mfma_dq_d##D_##_w##NW_,                                                    \
                   split.groups == 1   ? bwd_mfma_dkdv_d##D_##_w##NW_                             \
                   : split.groups == 4 ? bwd_mfma_dkdv_d##D_##_##FOUR_GROUPS                      \
                   : split.waves == 4  ? bwd_mfma_dkdv_d##D_##_##FOUR_WAVES                       \
                                       : bwd_mfma_dkdv_d##D_##_w##NW_##_split2);
    // (the last two columns: a kernel that the rule does not name there is not launched)
    BSA_LAUNCH(64, 2, w2_split4, w2_split2)
    BSA_LAUNCH(64, 4, w4_split4, w4_split2)
    BSA_LAUNCH(64, 8, w8_split4, w8_split2)
    BSA_LAUNCH(128, 4, w4_split2, w4_split2)
    BSA_LAUNCH(128, 8, w8_split2, w8_split2_wide)
#undef BSA_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace bsa
