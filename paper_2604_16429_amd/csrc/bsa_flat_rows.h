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

}  // namespace bsa
