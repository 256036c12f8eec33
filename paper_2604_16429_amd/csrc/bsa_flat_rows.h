// Walking the tokens of a list of blocks as one flat sequence (gfx950).
//
// The general-shape kernels take any tile: b tokens, any width.  The tokens of
// the listed blocks, in list order and inside a block in in-tile order, form a
// sequence of (number of blocks) * b rows, which is cut into tiles of KT rows
// for the matrix cores without regard to block boundaries: only the last tile of
// the whole sequence has padding.  Two tables in LDS turn a position into a token:
// the first token of every listed block and the offset of every in-tile
// position; a lane keeps (block, in-tile position) of its rows and advances them
// by KT without a division.
#pragma once

#include "bsa_device.h"
#include "bsa_mfma_common.h"

namespace bsa {

constexpr int kListTable = 1024;           // listed blocks the LDS table holds

// LDS of both tables for the attended blocks of one query block (at most 8 KiB:
// b <= 1024)
inline size_t flat_table_bytes(const Geom& g)
{
    const int listed = g.n_select + 1;
    return sizeof(uint32_t) * (size_t)(g.block_tokens + (listed < kListTable ? listed : kListTable));
}

// Lane l: 16 bytes from src to LDS lds + 16 l (lds uniform); see load_lds_16.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_lds_16_at(const void* src, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(lds), "v"(src) : "memory", "m0");
}
__device__ __forceinline__ void load_lds_4_at(const void* src, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 :: "s"(lds), "v"(src) : "memory", "m0");
}
#pragma clang diagnostic pop

// Offset, from the first token of its block, of every in-tile position.
__device__ __forceinline__ void fill_position_table(const Geom& g, uint32_t* pos_s)
{
    for (int tau = threadIdx.x; tau < g.block_tokens; tau += blockDim.x) {
        const int rr = tau / g.block_w;
        pos_s[tau] = (uint32_t)(rr * g.grid_w + (tau - rr * g.block_w));
    }
}

__device__ __forceinline__ uint32_t block_first_token(const Geom& g, int beta)
{
    const int br = beta / g.blocks_per_row, bc = beta - br * g.blocks_per_row;
    return (uint32_t)(br * g.block_h * g.grid_w + bc * g.block_w);
}

// Position of one row in the flat sequence: listed block, in-tile position.
struct FlatRow {
    int blk, tau;
    __device__ __forceinline__ void start(int p, int b)
    {
        blk = p / b;
        tau = p - blk * b;
    }
    // step_q, step_r: quotient and remainder of the advance by b
    __device__ __forceinline__ void advance(int step_q, int step_r, int b)
    {
        blk += step_q;
        tau += step_r;
        if (tau >= b) { tau -= b; ++blk; }
    }
};

// Shape of a [KT rows] x [D channels] tile in LDS.  Rows are D elements; the
// 16-byte chunks of a row are XOR-swizzled by the row so that a row-fragment read
// (the same chunk of 8 consecutive rows) and the transposing bf16 read (a chunk
// pair of 4 aligned rows) are free of bank conflicts.  The swizzle is applied on
// the global side of the direct-to-LDS load.
template <typename T, int D>
struct FlatTile {
    static constexpr int ROW_BYTES = D * (int)sizeof(T);
    static constexpr int KT = sizeof(T) == 2 ? 64 : 32;         // rows
    static constexpr int TILE_BYTES = KT * ROW_BYTES;
    static constexpr int SLABS = TILE_BYTES / 1024;             // loads of 64 x 16 bytes
    static constexpr int RPS = 1024 / ROW_BYTES;                // rows per slab
    static constexpr int LPR = ROW_BYTES / 16;                  // lanes per row

    static __device__ __forceinline__ int swz(int row, int chunk)
    {
        if (ROW_BYTES == 64) {       // 4 chunks, two rows per 128 bytes of banks
            const int x = (row >> 1) & 3;
            return chunk ^ (((x & 1) << 1) | (x >> 1));
        }
        return chunk ^ (((row & 3) << 1) | ((row >> 2) & 1));
    }
};

// Two fp32 weights as bf16 pairs hi + lo: hi the upper 16 bits, lo the rounded
// rest, together 16 significant bits.
__device__ __forceinline__ void split_bf16(float a, float b, uint32_t& hi, uint32_t& lo)
{
    const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    hi = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
    lo = pack_bf16(a - __uint_as_float(ua & 0xffff0000u), b - __uint_as_float(ub & 0xffff0000u));
}

__device__ __forceinline__ f32x16 zero_tile()
{
    const f32x16 z = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f,
                      0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    return z;
}

// acc + X Y^T for 32 tile rows X and 32 stationary rows Y: this lane's column is
// its stationary row yf (bf16: B operands of the 16-channel steps; fp32: the
// channels 8 j + 4 half + 0..3), register r is tile row 8 (r/4) + 4 half + r%4.
template <int D>
__device__ __forceinline__ f32x16 dot_tile(const unsigned char* x_rows, const bf16x8 (&yf)[D / 16],
                                           f32x16 acc, int l32, int half)
{
    using Tile = FlatTile<uint16_t, D>;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        const bf16x8 xf = *(const bf16x8*)(x_rows + l32 * Tile::ROW_BYTES +
                                           Tile::swz(l32, 2 * ks + half) * 16);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, yf[ks], acc, 0, 0, 0);
    }
    return acc;
}
template <int D>
__device__ __forceinline__ f32x16 dot_tile(const unsigned char* x_rows, const float4 (&yf)[D / 8],
                                           f32x16 acc, int l32, int half)
{
    using Tile = FlatTile<float, D>;
#pragma unroll
    for (int j = 0; j < D / 8; ++j) {
        const float4 xf = *(const float4*)(x_rows + l32 * Tile::ROW_BYTES +
                                           Tile::swz(l32, 2 * j + half) * 16);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.x, yf[j].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.y, yf[j].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.z, yf[j].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xf.w, yf[j].w, acc, 0, 0, 0);
    }
    return acc;
}

// acc^T += X^T W^T for 32 tile rows X: channels x this lane's column; w: the
// column's weights of the 32 rows in the accumulator layout of dot_tile, which is
// the B operand as it stands.
template <int D>
__device__ __forceinline__ void weighted_rows(const uint16_t*, const unsigned char* x_rows,
                                              const f32x16& w, f32x16 (&acc)[D / 32], int lane)
{
    using Tile = FlatTile<uint16_t, D>;
    const int s16 = lane & 15, gq = lane >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            split_bf16(w[8 * h + 2 * e], w[8 * h + 2 * e + 1], hi[e], lo[e]);
        const bf16x8 w_hi = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
        const bf16x8 w_lo = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
            // transposing read: source lane s of 16-lane group gq supplies 8 bytes
            // of X[16 h + 8 rd + 4 (gq/2) + s/4][32 dt + 16 (gq%2) + 4 (s%4)]
            const int col = 16 * (gq & 1) + 4 * (s16 & 3) + 32 * dt;
            bf16x4 part[2];
#pragma unroll
            for (int rd = 0; rd < 2; ++rd) {
                const int row = 16 * h + 8 * rd + 4 * (gq >> 1) + (s16 >> 2);
                const unsigned char* src = x_rows + row * Tile::ROW_BYTES +
                                           Tile::swz(row, col >> 3) * 16 + (col & 7) * 2;
                part[rd] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, src));
            }
            const bf16x8 xf = __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
            acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, w_hi, acc[dt], 0, 0, 0);
            acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, w_lo, acc[dt], 0, 0, 0);
        }
    }
}
template <int D>
__device__ __forceinline__ void weighted_rows(const float*, const unsigned char* x_rows,
                                              const f32x16& w, f32x16 (&acc)[D / 32], int lane)
{
    using Tile = FlatTile<float, D>;
    const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * half + (r & 3);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
            const int chunk = 8 * dt + (l32 >> 2);
            const float x = *(const float*)(x_rows + row * Tile::ROW_BYTES +
                                            Tile::swz(row, chunk) * 16 + (l32 & 3) * 4);
            acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, w[r], acc[dt], 0, 0, 0);
        }
    }
}

__device__ __forceinline__ void load_row(const uint16_t* row, bf16x8& f, int step, int half)
{
    f = *(const bf16x8*)(row + 16 * step + 8 * half);
}
__device__ __forceinline__ void load_row(const float* row, float4& f, int step, int half)
{
    f = *(const float4*)(row + 8 * step + 4 * half);
}

// A stationary row as the operand of dot_tile: 16-byte pieces of the lane's half.
template <typename T, int D> struct RowFrag;
template <int D> struct RowFrag<uint16_t, D> { typedef bf16x8 type; static constexpr int N = D / 16; };
template <int D> struct RowFrag<float, D> { typedef float4 type; static constexpr int N = D / 8; };


// Padding of the last tile: register r of a 32-row tile with `left` rows is a row
// past the end.
__device__ __forceinline__ bool past_end(int r, int half, int left)
{
    return 8 * (r >> 2) + 4 * half + (r & 3) >= left;
}

__device__ __forceinline__ bf16x8 negated(bf16x8 x)
{
    uint4 u = __builtin_bit_cast(uint4, x);
    u.x ^= 0x80008000u; u.y ^= 0x80008000u; u.z ^= 0x80008000u; u.w ^= 0x80008000u;
    return __builtin_bit_cast(bf16x8, u);
}
__device__ __forceinline__ float4 negated(float4 x)
{
    return make_float4(-x.x, -x.y, -x.z, -x.w);
}

// Stores this lane's column of D channels (accumulators of weighted_rows), scaled
// by f, to its token row; with `extra` see store4_or_add.
template <typename T, int D>
__device__ __forceinline__ void store_column(T* row, const f32x16 (&acc)[D / 32], float f,
                                             const float* extra, float inv_b, int half)
{
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int d = 32 * dt + 8 * r4 + 4 * half;
            store4_or_add(row + d,
                          make_float4(acc[dt][4 * r4] * f, acc[dt][4 * r4 + 1] * f,
                                      acc[dt][4 * r4 + 2] * f, acc[dt][4 * r4 + 3] * f),
                          extra ? extra + d : nullptr, inv_b);
        }
}

// The keys that a query block attends to, as a flat sequence gathered tile by tile
// by the first NL wavefronts of a workgroup: block i itself followed by its
// selected blocks, or, when the lists stand alone (list_only), exactly the listed
// blocks.  Up to 63 listed blocks are visited in ascending order (query blocks
// that run together then sweep the slice's K/V in the same direction).
template <typename T, int D, int NL>
struct AttendedKeys {
    using Tile = FlatTile<T, D>;
    static constexpr int MINE = Tile::SLABS / NL;
    static_assert(Tile::SLABS % NL == 0, "slabs split evenly between the loading wavefronts");

    int total, tiles;               // keys, tiles
    int b, n, step_q, step_r, wave;
    const int32_t* sel_row;
    const uint32_t *pos_s, *first_s;
    FlatRow at[MINE];               // this lane's row of slab wave + NL j of the next tile
    uint32_t chunk_off[MINE];

    // Fills the LDS tables (flat_table_bytes); a barrier has to follow.
    __device__ __forceinline__ void init(const Geom& g, const int32_t* sel_idx, int64_t bh_idx,
                                         int i, uint32_t* tables_s, int lane, int wave_)
    {
        wave = wave_;
        b = g.block_tokens;
        uint32_t* pos = tables_s;                     // [b]
        uint32_t* blocks = tables_s + b;              // [min(listed blocks, kListTable)]
        pos_s = pos;
        first_s = blocks;
        const int list_only = g.list_only;
        sel_row = sel_idx + (bh_idx * g.n_blocks + i) * g.n_select + list_only;
        const int first = list_only ? sel_row[-1] : i;
        n = g.n_select - list_only;                   // blocks after the first
        fill_position_table(g, pos);
        if (n < 64) {
            if (wave == 0) {
                const int mine = lane < n ? sel_row[lane] : 0x7fffffff;
                int rank = 1;
                for (int t = 0; t < n; ++t)
                    rank += __builtin_amdgcn_readlane(mine, t) < mine ? 1 : 0;
                if (lane < n) blocks[rank] = block_first_token(g, mine);
                if (lane == 0) blocks[0] = block_first_token(g, first);
            }
        } else {
            for (int t = threadIdx.x; t <= n && t < kListTable; t += blockDim.x)
                blocks[t] = block_first_token(g, t == 0 ? first : sel_row[t - 1]);
        }
        geom = &g;
        total = (n + 1) * b;
        tiles = (total + Tile::KT - 1) / Tile::KT;
        step_q = Tile::KT / b;
        step_r = Tile::KT - step_q * b;
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int row = Tile::RPS * (wave + NL * j) + lane / Tile::LPR;
            at[j].start(row, b);
            chunk_off[j] = (uint32_t)Tile::swz(row, lane % Tile::LPR) * 16u;
        }
    }

    // Gathers the next tile of both tensors (kb, vb: their slices; k_dst, v_dst: LDS
    // addresses of the tiles) and moves on.  Rows past the end repeat the last row;
    // they carry no weight.
    __device__ __forceinline__ void gather_next(const unsigned char* kb, const unsigned char* vb,
                                                uint32_t k_dst, uint32_t v_dst)
    {
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const bool past = at[j].blk > n;
            const int blk = past ? n : at[j].blk, tau = past ? b - 1 : at[j].tau;
            const uint32_t org = blk < kListTable ? first_s[blk]
                                                  : block_first_token(*geom, sel_row[blk - 1]);
            const uint64_t off = (uint64_t)(org + pos_s[tau]) * Tile::ROW_BYTES + chunk_off[j];
            const uint32_t dst = (uint32_t)(wave + NL * j) * 1024u;
            load_lds_16_at(kb + off, k_dst + dst);
            load_lds_16_at(vb + off, v_dst + dst);
            at[j].advance(step_q, step_r, b);
        }
    }

private:
    const Geom* geom;
};

// Rows of a block over workgroups of at most `max_waves` wavefronts of 32 rows
// each: as few workgroups as hold them, as even as possible.
struct RowSplit {
    int chunks, waves;
    RowSplit(int block_tokens, int max_waves)
    {
        const int row_tiles = (block_tokens + 31) / 32;
        chunks = (row_tiles + max_waves - 1) / max_waves;
        waves = (row_tiles + chunks - 1) / chunks;
    }
};

}  // namespace bsa
