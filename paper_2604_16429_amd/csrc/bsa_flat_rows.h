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

#include <type_traits>

namespace bsa {

constexpr int kListTable = 1024;           // listed blocks the LDS table holds

// Entries behind the last listed block that repeat it: rows past the end of the last
// tile (of kt rows), and of the tile after it (split: the last of as many tiles), which is
// looked up but not gathered, then look up like any other row.  They carry no weight.
__host__ __device__ constexpr int repeated_entries(int kt, int b, int split = 1)
{
    return ((split + 1) * kt - 2) / b + 1;
}

// LDS of both tables for `listed` attended blocks (at most 9 KiB: b <= 1024)
inline size_t flat_table_bytes(const Geom& g, int listed, int split = 1, int kt = 64)
{
    return sizeof(uint32_t) *
           (size_t)(g.block_tokens + (listed < kListTable ? listed : kListTable) +
                    repeated_entries(kt, g.block_tokens, split));
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

// Position of one row in the flat sequence: listed block, in-tile position.  Both
// tables hold tokens, rows past the end need no test and the gathers take 32-bit
// offsets from a descriptor, so that a gathered row costs about 10 vector instructions
// (with clamped rows and 64-bit addresses 24: per 32 x 32 tile of the forward at head
// dim 64 146 instead of 153 instructions in all; fp32 training pass, 1.5 degree grid,
// 8 heads, 1.79 -> 1.74 ms, bf16 with tiles of 10 x 10 1.015 -> 1.006 ms).
struct FlatRow {
    uint32_t blk, tau;
    __device__ __forceinline__ void start(int p, int b)
    {
        blk = (uint32_t)p / (uint32_t)b;
        tau = (uint32_t)p - blk * (uint32_t)b;
    }
    // step_q, step_r: quotient and remainder of the advance by b
    __device__ __forceinline__ void advance(uint32_t step_q, uint32_t step_r, uint32_t b)
    {
        const uint32_t t = tau + step_r;
        blk += step_q + (t >= b ? 1u : 0u);
        tau = min(t, t - b);                 // t < b: t - b wraps to a large number
    }
};

// Rows gathered to LDS from `bytes` bytes at base, 16 bytes per lane.  Offsets are 32
// bits where the rows allow it (wide: they do not, and addresses are 64 bits).
struct RowSource {
    i32x4 rsrc;
    const unsigned char* base;
    bool wide;
    __device__ __forceinline__ RowSource(const void* p, int64_t bytes)
        : rsrc(buffer_desc(p, (uint32_t)bytes)), base((const unsigned char*)p),
          wide(bytes >= (int64_t)1 << 31)
    {
    }
};

// Shape of a [KT rows] x [D channels] tile in LDS.  Rows are D elements; the
// 16-byte chunks of a row are XOR-swizzled by the row so that a row-fragment read
// (the same chunk of 8 consecutive rows) and the transposing bf16 read (a chunk
// pair of 4 aligned rows) are free of bank conflicts.  The swizzle is applied on
// the global side of the direct-to-LDS load.
template <typename T, int D, int ROWS = sizeof(T) == 2 ? 64 : 32>
struct FlatTile {
    static constexpr int ROW_BYTES = D * (int)sizeof(T);
    static constexpr int KT = ROWS;
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

// What a wavefront holds of a 32-row tile against its own ROWS stationary rows (one per
// lane column, `col`): NR values per lane, value r of tile row
// STEP (r/4) + 4 part + r%4, part = lane / ROWS.
//   bf16: 32 stationary rows, v_mfma_f32_32x32x16_bf16.
//   fp32: 16, v_mfma_f32_16x16x4_f32: the same rate as 32x32x2 (64 operations per cycle
//         and SIMD) with half the registers, so that twice as many wavefronts share a
//         block: a chain of products that depend on each other is half as long, and four
//         (backward three) wavefronts per SIMD instead of two cover it.
//   Rows16: bf16 with 16, v_mfma_f32_16x16x32_bf16 (the same rate), for the last wavefront of
//         a block when it has no more rows than that: half the vector work and matrix
//         instructions, where 32 columns would be mostly idle.  Tiles of 10 x 10, whose
//         fourth wavefront has four rows, work 112 rows instead of 128.
struct Rows16 {};
template <typename T> struct WaveTile;
template <> struct WaveTile<Rows16> {
    static constexpr int ROWS = 16, NR = 8, STEP = 16;
    typedef __attribute__((ext_vector_type(8))) float vec;
};
template <> struct WaveTile<uint16_t> {
    static constexpr int ROWS = 32, NR = 16, STEP = 8;
    typedef f32x16 vec;
};
template <> struct WaveTile<float> {
    static constexpr int ROWS = 16, NR = 8, STEP = 16;
    typedef __attribute__((ext_vector_type(8))) float vec;
};
template <typename T>
__device__ __forceinline__ typename WaveTile<T>::vec constant_tile(float x)
{
    typename WaveTile<T>::vec v;
#pragma unroll
    for (int r = 0; r < WaveTile<T>::NR; ++r) v[r] = x;
    return v;
}
// Largest value and sum over the lanes that share a column.
template <typename T> __device__ __forceinline__ float column_max(float x)
{
    x = fmaxf(x, swap32(x));
    return WaveTile<T>::ROWS == 16 ? fmaxf(x, __shfl_xor(x, 16)) : x;
}
template <typename T> __device__ __forceinline__ float column_sum(float x)
{
    x += swap32(x);
    return WaveTile<T>::ROWS == 16 ? x + __shfl_xor(x, 16) : x;
}
// A column of D channels: the accumulators of weighted_rows.
template <typename T, int D> struct Column;
template <int D> struct Column<uint16_t, D> { f32x16 a[D / 32]; };
template <int D> struct Column<float, D> { f32x4 a[D / 16]; };
template <int D> struct Column<Rows16, D> { f32x4 a[D / 16]; };
template <typename T, int D>
__device__ __forceinline__ void scale_column(Column<T, D>& c, float f)
{
#pragma unroll
    for (auto& a : c.a) a *= f;
}
template <typename T, int D> __device__ __forceinline__ void clear_column(Column<T, D>& c)
{
#pragma unroll
    for (auto& a : c.a) a = 0.0f;
}
// Where a lane reads a 32-row tile in LDS.  The swizzle leaves few distinct
// addresses per lane: everything else is a constant that goes into the read's
// offset field.  (Written out because the compiler otherwise keeps an address register
// per read, which does not fit beside the rest: it spills them, and a reload from
// scratch memory waits for every gather in flight.)
template <typename T, int D> struct TileReader;

template <int D> struct TileReader<uint16_t, D> {
    using Tile = FlatTile<uint16_t, D>;
    static constexpr int STEPS = D / 16, BASES = STEPS < 4 ? STEPS : 4;
    static constexpr int WBASES = D == 32 ? 1 : 2;
    uint32_t row[BASES];        // chunk 2 s + half of row l32, s < BASES
    uint32_t trans[WBASES];     // transposing read of channels 32 dt, dt < WBASES
    __device__ __forceinline__ void init(int lane)
    {
        const int l32 = lane & 31, half = lane >> 5, s16 = lane & 15, gq = lane >> 4;
#pragma unroll
        for (int s = 0; s < BASES; ++s)
            row[s] = (uint32_t)(l32 * Tile::ROW_BYTES + Tile::swz(l32, 2 * s + half) * 16);
        // source lane s16 of 16-lane group gq supplies 8 bytes of row
        // 4 (gq/2) + s16/4 (+ 16 h + 8 rd), channel 16 (gq%2) + 4 (s16%4) + 32 dt
        const int r = 4 * (gq >> 1) + (s16 >> 2);
#pragma unroll
        for (int dt = 0; dt < WBASES; ++dt) {
            const int col = 16 * (gq & 1) + 4 * (s16 & 3) + 32 * dt;
            trans[dt] = (uint32_t)(r * Tile::ROW_BYTES + Tile::swz(r, col >> 3) * 16 + (col & 7) * 2);
        }
    }
};
template <int D> struct TileReader<float, D> {
    using Tile = FlatTile<float, D>;
    static constexpr int BASES = 2;
    uint32_t row[BASES];        // chunk 4 s + part of row col, s < 2
    uint32_t col[4];            // row 4 part + r, r < 4, channels VEC col ..
    static constexpr int VEC = D == 32 ? 2 : 4;
    __device__ __forceinline__ void init(int lane)
    {
        const int c16 = lane & 15, part = lane >> 4;
#pragma unroll
        for (int s = 0; s < BASES; ++s)
            row[s] = (uint32_t)(c16 * Tile::ROW_BYTES + Tile::swz(c16, 4 * s + part) * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rr = 4 * part + r, at = 4 * VEC * c16;
            col[r] = (uint32_t)(rr * Tile::ROW_BYTES + Tile::swz(rr, at >> 4) * 16 + (at & 15));
        }
    }
};
template <int D> struct TileReader<Rows16, D> {
    using Tile = FlatTile<uint16_t, D>;
    static constexpr int BASES = D == 32 ? 1 : 2, WBASES = D == 32 ? 2 : 4;
    uint32_t row[BASES];        // chunk 4 s + part of row col, s < BASES
    uint32_t trans[WBASES];     // transposing read of channels 16 ct, ct < WBASES
    __device__ __forceinline__ void init(int lane)
    {
        const int c16 = lane & 15, part = lane >> 4;
#pragma unroll
        for (int s = 0; s < BASES; ++s)
            row[s] = (uint32_t)(c16 * Tile::ROW_BYTES + Tile::swz(c16, 4 * s + part) * 16);
        // source lane c16 of 16-lane group `part` supplies 8 bytes of row 4 part + c16/4
        // (+ 16), channel 4 (c16%4) + 16 ct
        const int r = 4 * part + (c16 >> 2);
#pragma unroll
        for (int ct = 0; ct < WBASES; ++ct) {
            const int at = 4 * (c16 & 3) + 16 * ct;
            trans[ct] = (uint32_t)(r * Tile::ROW_BYTES + Tile::swz(r, at >> 3) * 16 + (at & 7) * 2);
        }
    }
};

// Products of a 32-row tile.  LDS reads are issued a group ahead of the matrix
// instructions that use them, and held there (sched_barrier): the compiler would
// reuse one group's registers and expose the read latency between groups.
//
// Row products, acc + X Y^T: this lane's column is its stationary row (y: its
// pieces).  A piece is 16 channels: in bf16 channels 16 s + 8 part + 0..7 of each lane,
// one instruction; in fp32 16 s + 4 part + 0..3, four instructions for each of the two
// 16-row halves of the tile.
template <typename T, int D> struct RowPieces;
template <int D> struct RowPieces<uint16_t, D> {
    typedef bf16x8 type, frag;
    static constexpr int N = D / 16, GROUP = N < 4 ? N : 4;
};
struct RowFrag16 {
    f32x4 t[2];
};
// (Rows16: a piece is 32 channels, 32 s + 8 part + 0..7 of each lane, one instruction for
// each of the two 16-row halves)
struct RowFragBf16 {
    bf16x8 t[2];
};
template <int D> struct RowPieces<Rows16, D> {
    typedef bf16x8 type;
    typedef RowFragBf16 frag;
    static constexpr int N = D / 32, GROUP = N;
};
template <int D> struct RowPieces<float, D> {
    typedef f32x4 type;
    typedef RowFrag16 frag;
    static constexpr int N = D / 16, GROUP = 1;
};

template <int D>
__device__ __forceinline__ void read_rows(const TileReader<uint16_t, D>& rd, uint32_t tile, int imm,
                                          int group, bf16x8 (&x)[RowPieces<uint16_t, D>::GROUP])
{
#pragma unroll
    for (int u = 0; u < RowPieces<uint16_t, D>::GROUP; ++u) {
        const int s = group * RowPieces<uint16_t, D>::GROUP + u;
        x[u] = lds_read<bf16x8>(rd.row[s % rd.BASES] + tile, imm + (s / rd.BASES) * 128);
    }
}
template <int D>
__device__ __forceinline__ void read_rows(const TileReader<float, D>& rd, uint32_t tile, int imm,
                                          int group, RowFrag16 (&x)[RowPieces<float, D>::GROUP])
{
#pragma unroll
    for (int u = 0; u < RowPieces<float, D>::GROUP; ++u) {
        const int s = group * RowPieces<float, D>::GROUP + u;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            x[u].t[t] = lds_read<f32x4>(rd.row[s % rd.BASES] + tile,
                                        imm + (s / rd.BASES) * 128 + 16 * t * FlatTile<float, D>::ROW_BYTES);
    }
}
template <int D>
__device__ __forceinline__ void read_rows(const TileReader<Rows16, D>& rd, uint32_t tile, int imm,
                                          int, RowFragBf16 (&x)[RowPieces<Rows16, D>::GROUP])
{
#pragma unroll
    for (int s = 0; s < RowPieces<Rows16, D>::GROUP; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t)
            x[s].t[t] = lds_read<bf16x8>(rd.row[s % rd.BASES] + tile,
                                         imm + (s / rd.BASES) * 128 + 16 * t * 2 * D);
}
typedef WaveTile<float>::vec f32x8;
__device__ __forceinline__ f32x4 half_tile(const f32x8& v, int t)
{
    return t ? __builtin_shufflevector(v, v, 4, 5, 6, 7) : __builtin_shufflevector(v, v, 0, 1, 2, 3);
}
__device__ __forceinline__ f32x16 mul_piece(bf16x8 x, bf16x8 y, f32x16 acc)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, acc, 0, 0, 0);
}
__device__ __forceinline__ f32x8 mul_piece(const RowFrag16& x, f32x4 y, f32x8 acc)
{
    f32x4 a = half_tile(acc, 0), b = half_tile(acc, 1);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        a = __builtin_amdgcn_mfma_f32_16x16x4f32(x.t[0][c], y[c], a, 0, 0, 0);
        b = __builtin_amdgcn_mfma_f32_16x16x4f32(x.t[1][c], y[c], b, 0, 0, 0);
    }
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ f32x8 mul_piece(const RowFragBf16& x, bf16x8 y, f32x8 acc)
{
    const f32x4 a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.t[0], y, half_tile(acc, 0), 0, 0, 0);
    const f32x4 b = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.t[1], y, half_tile(acc, 1), 0, 0, 0);
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// acc + X Y^T.  tile: LDS address of the tile (uniform), imm: constant to add.
template <typename T, int D>
__device__ __forceinline__ typename WaveTile<T>::vec dot_tile(
    const TileReader<T, D>& rd, uint32_t tile, int imm,
    const typename RowPieces<T, D>::type (&y)[RowPieces<T, D>::N], typename WaveTile<T>::vec acc)
{
    constexpr int G = RowPieces<T, D>::GROUP, GROUPS = RowPieces<T, D>::N / G;
    typename RowPieces<T, D>::frag x[2][G];
    read_rows(rd, tile, imm, 0, x[0]);
#pragma unroll
    for (int gr = 0; gr < GROUPS; ++gr) {
        if (gr + 1 < GROUPS) read_rows(rd, tile, imm, gr + 1, x[(gr + 1) & 1]);
        if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < G; ++u) acc = mul_piece(x[gr & 1][u], y[gr * G + u], acc);
        if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
}
// Two row products side by side (two independent accumulation chains).  APART, fp32 at
// 64 and 128 channels: the first product in four chains, summed one by one.  A score
// that is one chain of 128 products is rounded twice as far as four of 32, and its
// weight carries that into dV and dK (scores of 22 whose terms have one sign: 3.5e-6
// against 1.6e-6 of them; fp32 training passes 0.3 to 1.3 % longer).
template <bool APART, typename T, int D>
__device__ __forceinline__ void dot_tiles(
    const TileReader<T, D>& rd, uint32_t tile_a, uint32_t tile_b, int imm,
    const typename RowPieces<T, D>::type (&ya)[RowPieces<T, D>::N],
    const typename RowPieces<T, D>::type (&yb)[RowPieces<T, D>::N], typename WaveTile<T>::vec& acc_a,
    typename WaveTile<T>::vec& acc_b)
{
    constexpr int G = RowPieces<T, D>::GROUP, N = RowPieces<T, D>::N, GROUPS = N / G;
    constexpr int CHAIN = APART && sizeof(T) == 4 && D > 32 ? N / 4 : N;     // pieces
    typename RowPieces<T, D>::frag a[2][G], b[2][G];
    read_rows(rd, tile_a, imm, 0, a[0]);
    read_rows(rd, tile_b, imm, 0, b[0]);
    typename WaveTile<T>::vec chain = acc_a;
#pragma unroll
    for (int gr = 0; gr < GROUPS; ++gr) {
        if (gr + 1 < GROUPS) {
            read_rows(rd, tile_a, imm, gr + 1, a[(gr + 1) & 1]);
            read_rows(rd, tile_b, imm, gr + 1, b[(gr + 1) & 1]);
        }
        if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int piece = gr * G + u;
            if (piece > 0 && piece % CHAIN == 0) chain = constant_tile<T>(0.0f);
            chain = mul_piece(a[gr & 1][u], ya[piece], chain);
            acc_b = mul_piece(b[gr & 1][u], yb[piece], acc_b);
            if ((piece + 1) % CHAIN == 0) acc_a = piece < CHAIN ? chain : acc_a + chain;
        }
        if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
    }
}

// Weighted row sums, acc^T += X^T W^T: channels x this lane's column; w: the
// column's weights of the 32 rows in the accumulator layout of dot_tile, which is
// the B operand as it stands.  Groups of 16 rows in bf16, of eight instructions in fp32;
// the caller reads group 0 (read_columns) before it computes the weights.
// fp32: the operand of output tile c is channel VEC col + c % VEC (+ 64 for c >= 4), so
// that one 16-byte read (8 at head dim 32) feeds four (two) instructions, and a lane ends
// up with consecutive channels of its column.
template <typename T, int D> struct ColumnPieces;
template <int D> struct ColumnPieces<uint16_t, D> {
    static constexpr int GROUPS = 2;
    bf16x8 x[D / 32];                       // A operand: channels 32 dt .. x 16 rows
};
template <int D> struct ColumnPieces<Rows16, D> {
    static constexpr int GROUPS = 1;
    bf16x8 x[D / 16];                       // A operand: channels 16 ct .. x 32 rows
};
template <int D> struct ColumnPieces<float, D> {
    static constexpr int VEC = TileReader<float, D>::VEC;
    typedef __attribute__((ext_vector_type(VEC))) float vec;
    static constexpr int STEPS = 128 / D, GROUPS = 8 / STEPS;
    vec x[STEPS][D / (16 * VEC)];           // row 16 (step / 4) + 4 part + step % 4
};
template <int D>
__device__ __forceinline__ void read_columns(const TileReader<uint16_t, D>& rd, uint32_t tile, int imm,
                                             int group, ColumnPieces<uint16_t, D>& c)
{
    constexpr int ROW = FlatTile<uint16_t, D>::ROW_BYTES;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
        bf16x4 part[2];
#pragma unroll
        for (int r = 0; r < 2; ++r)
            part[r] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                (__attribute__((address_space(3))) bf16x4*)(uintptr_t)(
                    rd.trans[dt % rd.WBASES] + tile +
                    (uint32_t)(imm + (16 * group + 8 * r) * ROW + (dt / rd.WBASES) * 128)));
        c.x[dt] = __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
    }
}
// (rows 4 part + 0..3 and 16 + 4 part + 0..3: the order in which a lane holds its weights)
template <int D>
__device__ __forceinline__ void read_columns(const TileReader<Rows16, D>& rd, uint32_t tile, int imm,
                                             int, ColumnPieces<Rows16, D>& c)
{
#pragma unroll
    for (int ct = 0; ct < D / 16; ++ct) {
        bf16x4 part[2];
#pragma unroll
        for (int r = 0; r < 2; ++r)
            part[r] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                (__attribute__((address_space(3))) bf16x4*)(uintptr_t)(
                    rd.trans[ct % rd.WBASES] + tile +
                    (uint32_t)(imm + 16 * r * 2 * D + (ct / rd.WBASES) * 128)));
        c.x[ct] = __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
    }
}
template <int D>
__device__ __forceinline__ void read_columns(const TileReader<float, D>& rd, uint32_t tile, int imm,
                                             int group, ColumnPieces<float, D>& c)
{
    constexpr int ROW = FlatTile<float, D>::ROW_BYTES;
    typedef typename ColumnPieces<float, D>::vec V;
#pragma unroll
    for (int u = 0; u < c.STEPS; ++u) {
        const int step = c.STEPS * group + u;
#pragma unroll
        for (int e = 0; e < D / (16 * c.VEC); ++e)
            c.x[u][e] = lds_read<V>(rd.col[step & 3] + tile, imm + 16 * (step >> 2) * ROW + 256 * e);
    }
}
template <int D>
__device__ __forceinline__ void add_columns(const ColumnPieces<uint16_t, D>& c, const f32x16& w,
                                            int group, Column<uint16_t, D>& acc)
{
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        split_bf16(w[8 * group + 2 * e], w[8 * group + 2 * e + 1], hi[e], lo[e]);
    const bf16x8 w_hi = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
    const bf16x8 w_lo = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
        acc.a[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c.x[dt], w_hi, acc.a[dt], 0, 0, 0);
        acc.a[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c.x[dt], w_lo, acc.a[dt], 0, 0, 0);
    }
}
template <int D>
__device__ __forceinline__ void add_columns(const ColumnPieces<Rows16, D>& c, const f32x8& w, int,
                                            Column<Rows16, D>& acc)
{
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split_bf16(w[2 * e], w[2 * e + 1], hi[e], lo[e]);
    const bf16x8 w_hi = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
    const bf16x8 w_lo = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
#pragma unroll
    for (int ct = 0; ct < D / 16; ++ct) {
        acc.a[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c.x[ct], w_hi, acc.a[ct], 0, 0, 0);
        acc.a[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c.x[ct], w_lo, acc.a[ct], 0, 0, 0);
    }
}
template <int D>
__device__ __forceinline__ void add_columns(const ColumnPieces<float, D>& c, const f32x8& w, int group,
                                            Column<float, D>& acc)
{
#pragma unroll
    for (int u = 0; u < c.STEPS; ++u)
#pragma unroll
        for (int t = 0; t < D / 16; ++t)
            acc.a[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                c.x[u][t / c.VEC][t % c.VEC], w[c.STEPS * group + u], acc.a[t], 0, 0, 0);
}
template <typename T, int D>
__device__ __forceinline__ void weighted_rows(const TileReader<T, D>& rd, uint32_t tile, int imm,
                                              ColumnPieces<T, D>& first,
                                              const typename WaveTile<T>::vec& w, Column<T, D>& acc)
{
    constexpr int GROUPS = ColumnPieces<T, D>::GROUPS;
    ColumnPieces<T, D> second;
#pragma unroll
    for (int gr = 0; gr < GROUPS; ++gr) {
        ColumnPieces<T, D>&cur = gr & 1 ? second : first, &nxt = gr & 1 ? first : second;
        if (gr + 1 < GROUPS) read_columns(rd, tile, imm, gr + 1, nxt);
        if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
        add_columns(cur, w, gr, acc);
        if (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
    }
}

// Piece `step` of a stationary row.  K: the key of the row pieces (element type or Rows16).
template <typename K>
__device__ __forceinline__ void load_row(const uint16_t* row, bf16x8& f, int step, int part)
{
    f = *(const bf16x8*)(row + (std::is_same<K, Rows16>::value ? 32 : 16) * step + 8 * part);
}
template <typename K>
__device__ __forceinline__ void load_row(const float* row, f32x4& f, int step, int part)
{
    f = *(const f32x4*)(row + 16 * step + 4 * part);
}

// Padding of the last tile: value r of a 32-row tile with `left` rows is a row past the
// end.
template <typename T> __device__ __forceinline__ bool past_end(int r, int part, int left)
{
    return WaveTile<T>::STEP * (r >> 2) + 4 * part + (r & 3) >= left;
}

__device__ __forceinline__ f32x4 negated(f32x4 x)
{
    return -x;
}

// Stores this lane's column of D channels, scaled by f, to its token row; with `extra`
// see store4_or_add.
template <int D>
__device__ __forceinline__ void store_column(uint16_t* row, const Column<uint16_t, D>& acc, float f,
                                             const float* extra, float inv_b, int part)
{
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int d = 32 * dt + 8 * r4 + 4 * part;
            const f32x16& a = acc.a[dt];
            store4_or_add(row + d,
                          make_float4(a[4 * r4] * f, a[4 * r4 + 1] * f, a[4 * r4 + 2] * f,
                                      a[4 * r4 + 3] * f),
                          extra ? extra + d : nullptr, inv_b);
        }
}
template <int D>
__device__ __forceinline__ void store_column(uint16_t* row, const Column<Rows16, D>& acc, float f,
                                             const float* extra, float inv_b, int part)
{
#pragma unroll
    for (int ct = 0; ct < D / 16; ++ct) {
        const int d = 16 * ct + 4 * part;
        const f32x4& a = acc.a[ct];
        store4_or_add(row + d, make_float4(a[0] * f, a[1] * f, a[2] * f, a[3] * f),
                      extra ? extra + d : nullptr, inv_b);
    }
}
// (value r of output tile c is channel VEC (4 part + r) + c % VEC, + 64 for c >= 4)
template <int D>
__device__ __forceinline__ void store_column(float* row, const Column<float, D>& acc, float f,
                                             const float* extra, float inv_b, int part)
{
    constexpr int VEC = TileReader<float, D>::VEC;
    auto value = [&](int d) {                         // channel VEC 4 part + d of its 64
        return acc.a[d / (4 * VEC) * VEC + d % VEC][d % (4 * VEC) / VEC] * f;
    };
#pragma unroll
    for (int d = 0; d < D / 4; d += 4) {
        const int at = 64 * (d / 16) + 4 * VEC * part + d % 16;
        store4_or_add(row + at,
                      make_float4(value(d), value(d + 1), value(d + 2), value(d + 3)),
                      extra ? extra + at : nullptr, inv_b);
    }
}

// This wavefront's share of a tile of two tensors: slabs wave + NL j, row tok[j] of
// both (ks and vs are equally long).
template <typename Tile, int MINE, int NL>
__device__ __forceinline__ void gather_rows(const RowSource& ks, const RowSource& vs,
                                            const uint32_t (&tok)[MINE],
                                            const uint32_t (&chunk_off)[MINE], int wave,
                                            uint32_t k_dst, uint32_t v_dst)
{
    if (__builtin_expect(!ks.wide, 1)) {
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const uint32_t off = tok[j] * (uint32_t)Tile::ROW_BYTES | chunk_off[j];
            const uint32_t dst = (uint32_t)(wave + NL * j) * 1024u;
            load_lds_16(ks.rsrc, off, 0u, k_dst + dst);
            load_lds_16(vs.rsrc, off, 0u, v_dst + dst);
        }
    } else {
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const uint64_t off = (uint64_t)tok[j] * Tile::ROW_BYTES + chunk_off[j];
            const uint32_t dst = (uint32_t)(wave + NL * j) * 1024u;
            load_lds_16_at(ks.base + off, k_dst + dst);
            load_lds_16_at(vs.base + off, v_dst + dst);
        }
    }
}

// The keys that a query block attends to, as a flat sequence gathered tile by tile
// by the first NL wavefronts of a workgroup: block i itself followed by its
// selected blocks, or, when the lists stand alone (list_only), exactly the listed
// blocks.  Up to 63 listed blocks are visited in ascending order (query blocks
// that run together then sweep the slice's K/V in the same direction).  SPLIT: as many
// groups of wavefronts take the tiles in turn, `wave` counts inside a group.
template <typename T, int D, int NL, int SPLIT = 1, class Tile_ = FlatTile<T, D>>
struct AttendedKeys {
    using Tile = Tile_;
    static constexpr int MINE = Tile::SLABS / NL;
    static_assert(Tile::SLABS % NL == 0, "slabs split evenly between the loading wavefronts");

    int total, tiles;               // keys, tiles
    int b, n, wave;
    uint32_t step_q, step_r;
    const int32_t* sel_row;
    const uint32_t *pos_s, *first_s;
    FlatRow at[MINE];               // this lane's row of slab wave + NL j of the tile after
    uint32_t tok[MINE];             // token of its row of the next tile
    uint32_t chunk_off[MINE];

    // Fills the LDS tables (flat_table_bytes); a barrier has to follow.
    __device__ __forceinline__ void init(const Geom& g, const int32_t* sel_idx, int64_t bh_idx,
                                         int i, uint32_t* tables_s, int lane, int wave_,
                                         int group = 0)
    {
        wave = wave_;
        b = g.block_tokens;
        uint32_t* pos = tables_s;                     // [b]
        uint32_t* blocks = tables_s + b;              // [min(listed blocks, kListTable) + repeats]
        pos_s = pos;
        first_s = blocks;
        const int list_only = g.list_only;
        sel_row = sel_idx + (bh_idx * g.n_blocks + i) * g.n_select + list_only;
        const int first = list_only ? sel_row[-1] : i;
        n = g.n_select - list_only;                   // blocks after the first
        fill_position_table(g, pos);
        const int repeats = repeated_entries(Tile::KT, b, SPLIT);
        if (n < 64) {
            if (wave == 0) {
                const int mine = lane < n ? sel_row[lane] : 0x7fffffff;
                int rank = 1;
                for (int t = 0; t < n; ++t) {
                    const int other = __builtin_amdgcn_readlane(mine, t);
                    rank += other < mine || (other == mine && t < lane) ? 1 : 0;
                }
                if (lane < n) {
                    const uint32_t tok0 = block_first_token(g, mine);
                    blocks[rank] = tok0;
                    if (rank == n)
                        for (int e = 1; e <= repeats; ++e) blocks[n + e] = tok0;
                }
                if (lane == 0) {
                    const uint32_t tok0 = block_first_token(g, first);
                    blocks[0] = tok0;
                    if (n == 0)
                        for (int e = 1; e <= repeats; ++e) blocks[e] = tok0;
                }
            }
        } else {
            const int table = min(n + 1 + repeats, kListTable);
            for (int t = threadIdx.x; t < table; t += blockDim.x)
                blocks[t] = block_first_token(g, t == 0 ? first : sel_row[min(t, n) - 1]);
        }
        geom = &g;
        total = (n + 1) * b;
        tiles = (total + Tile::KT - 1) / Tile::KT;
        step_q = (uint32_t)(SPLIT * Tile::KT / b);
        step_r = (uint32_t)(SPLIT * Tile::KT % b);
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int row = Tile::RPS * (wave + NL * j) + lane / Tile::LPR;
            at[j].start(Tile::KT * group + row, b);
            chunk_off[j] = (uint32_t)Tile::swz(row, lane % Tile::LPR) * 16u;
        }
    }

    // Looks up the rows of the next tile and moves on: once after the barrier, then
    // from gather_next, i.e. a whole tile before the tokens are used.  Rows past the
    // end take rows of the last block; they carry no weight.
    __device__ __forceinline__ void look_up()
    {
        if (n + 1 + repeated_entries(Tile::KT, b, SPLIT) <= kListTable) {
#pragma unroll
            for (int j = 0; j < MINE; ++j) {
                tok[j] = first_s[at[j].blk] + pos_s[at[j].tau];
                at[j].advance(step_q, step_r, b);
            }
        } else {                                      // long lists: the rest from the selection
#pragma unroll
            for (int j = 0; j < MINE; ++j) {
                const int blk = min((int)at[j].blk, n);
                tok[j] = (blk < kListTable ? first_s[blk]
                                           : block_first_token(*geom, sel_row[blk - 1])) +
                         pos_s[at[j].tau];
                at[j].advance(step_q, step_r, b);
            }
        }
    }

    // Gathers the next tile of both tensors (ks, vs: their slices; k_dst, v_dst: LDS
    // addresses of the tiles).
    __device__ __forceinline__ void gather_next(const RowSource& ks, const RowSource& vs,
                                                uint32_t k_dst, uint32_t v_dst)
    {
        gather_rows<Tile, MINE, NL>(ks, vs, tok, chunk_off, wave, k_dst, v_dst);
        look_up();
    }

private:
    const Geom* geom;
};

// Runs body(key) with the row pieces that a wavefront of `rows` rows takes.  MIXED: the
// kernel has the narrow form too (a kernel of its own: both forms in one took up to 3.5 %
// longer where no wavefront is narrow).
// `rows` is the same for all lanes of a wavefront, but not for all wavefronts of a workgroup: the
// narrow one runs its own copy of the body, workgroup barriers included.  That is sound on this
// hardware only, whose s_barrier counts the wavefronts that arrive, wherever they do, and only as
// long as both copies pass the same barriers in the same order: the body must not have a barrier,
// a return before one, or a trip count of a loop with one that depends on the key or on the rows.
template <typename K> struct PieceKey {
    typedef K type;
};
template <typename T, bool MIXED, class F> __device__ __forceinline__ void with_rows(int rows, F body)
{
    if constexpr (MIXED && sizeof(T) == 2) {
        if (rows <= 16) {
            body(PieceKey<Rows16>{});
            return;
        }
    }
    body(PieceKey<T>{});
}

// Rows of a block over workgroups of at most `max_waves` wavefronts of `rows` rows
// each: as few workgroups as hold them, as even as possible.
struct RowSplit {
    int chunks, waves;
    bool narrow;                // bf16: a wavefront has at most 16 of its 32 rows
    RowSplit(int block_tokens, int max_waves, int rows)
    {
        const int row_tiles = (block_tokens + rows - 1) / rows;
        chunks = (row_tiles + max_waves - 1) / max_waves;
        waves = (row_tiles + chunks - 1) / chunks;
        narrow = rows == 32 && chunks * waves * 32 - block_tokens >= 16;
    }
};

}  // namespace bsa
