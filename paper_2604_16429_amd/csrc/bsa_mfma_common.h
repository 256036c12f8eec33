// Pieces shared by the MFMA attention kernels (gfx950): operand vector types,
// the lane-32 exchange, the bf16 packing of the attention weights and the
// weights of one 32-key x 32-query tile.
#pragma once

#include "bsa_device.h"

namespace bsa {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

typedef __attribute__((ext_vector_type(4))) int32_t i32x4;

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

// Direct-to-LDS loads that the compiler does not track.  It orders every LDS
// read behind all direct-to-LDS loads that may have written the same object, so
// a double-buffered tile in one array costs a wait for the NEXT tile's loads in
// front of the current tile's first read.  These forms are for kernels that
// place the waits themselves: s_waitcnt vmcnt before the barrier that publishes
// the tile (the loads complete in order; the compiler's own waits can only be
// stricter for not knowing them).
// Buffer descriptor of `bytes` bytes at p (raw, bounds-checked: reads past the
// end return zeros).
__device__ __forceinline__ i32x4 buffer_desc(const void* p, uint32_t bytes)
{
    const uint64_t a = (uint64_t)p;
    const i32x4 d = {(int32_t)(uint32_t)a, (int32_t)((uint32_t)(a >> 32) & 0xffffu),
                     (int32_t)bytes, 0x00020000};
    return d;
}
// Byte address of an LDS object inside the workgroup's allocation.
__device__ __forceinline__ uint32_t lds_address(const void* p)
{
    return (uint32_t)(uintptr_t)LDS_PTR(void, p);
}
// (M0 holds the LDS address; the compiler warns that it may not preserve such a
// register, which is the point of naming it.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// Lane l: 16 bytes from rsrc[voff + soff] to LDS lds + 16 l (lds, soff uniform).
__device__ __forceinline__ void load_lds_16(i32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
// Lane l: 4 bytes from rsrc[voff + soff] to LDS lds + 4 l.
__device__ __forceinline__ void load_lds_4(i32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop

// Waits for this wavefront's direct-to-LDS loads in a form that the compiler
// accounts for: it then knows that loads it issued itself are done as well and
// does not wait for them (and for the gathers issued since) inside the loop.
__device__ __forceinline__ void wait_gathers()
{
    __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0)
}
// The same, and for its LDS reads (of a tile that is about to be overwritten).
__device__ __forceinline__ void wait_gathers_and_reads()
{
    __builtin_amdgcn_s_waitcnt(0x0070);     // vmcnt(0) lgkmcnt(0)
}

// 16 (or sizeof(V)) bytes from LDS byte address addr + imm: the constant goes into the
// read's offset field.
template <typename V>
__device__ __forceinline__ V lds_read(uint32_t addr, int imm)
{
    return *(const __attribute__((address_space(3))) V*)(uintptr_t)(addr + (uint32_t)imm);
}

// Exchange with the lane 32 away (lanes l < 32 get the value of l + 32 and
// vice versa).
__device__ __forceinline__ float swap32(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    // r[0] holds, for lanes < 32, their own value and for lanes >= 32 the value
    // of lane - 32; r[1] the opposite halves.
    return __uint_as_float(threadIdx.x & 32 ? r[0] : r[1]);
}

__device__ __forceinline__ bf16x8 negated(bf16x8 x)
{
    uint4 u = __builtin_bit_cast(uint4, x);
    u.x ^= 0x80008000u; u.y ^= 0x80008000u; u.z ^= 0x80008000u; u.w ^= 0x80008000u;
    return __builtin_bit_cast(bf16x8, u);
}

// P^T = exp2(S^T c2 - m_ref) for one 32-key x 32-query tile, rounded to bf16 B
// operands; returns this lane's sum of the fp32 weights.  Only builtins touch
// the MFMA results (never inline asm): the compiler must see these reads to
// place the wait states the hardware requires.
__device__ __forceinline__ float tile_weights(const f32x16& s, float c2, float neg_m,
                                              bf16x8 (&p)[2])
{
    float rs = 0.0f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(s[8 * h + 2 * e], c2, neg_m));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(s[8 * h + 2 * e + 1], c2, neg_m));
            w[e] = pack_bf16(p0, p1);
            rs += p0 + p1;
        }
        p[h] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
    }
    return rs;
}

constexpr float kSumLimit = 4096.0f;

// Orders a wavefront's LDS writes before reads by other lanes of it, and the other way
// round: the hardware keeps the order by itself, the compiler, which sees one lane's
// addresses and types, has to be told.  No instruction.
__device__ __forceinline__ void lane_exchange()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Stores a wavefront's 32 rows of D channels, bf16 (accumulators of transposed products:
// lane l32 of both halves holds row l32, register 4 r + e of tile dt channel 32 dt + 8 r +
// 4 half + e), scaled by f, to the in-tile positions pos0 .. pos0 + 31 of the block whose
// first token's row is `block`.  Tile width a power of two.  The rows go through 4 KiB of
// LDS (one per wavefront, nobody else's), 64 channels at a time and swizzled in 16-byte
// chunks, so that a store instruction writes runs of 128 bytes and more: straight from
// the accumulators it writes 8 bytes of 64 places.  Forward at head dim 64 (same form):
// 24 members at 1.5 degrees 4.47 -> 4.34 ms with the selection, one member 82.6 -> 79.6
// us, 0.25 degrees 20.98 -> 20.76 ms.
template <int D>
__device__ __forceinline__ void store_rows(uint16_t* block, const Geom& g, int pos0,
                                           const f32x16 (&acc)[D / 32], float f, unsigned char* lds,
                                           int lane)
{
    const int l32 = lane & 31, half = lane >> 5;
    const int shift = __builtin_ctz((unsigned)g.block_w);
    auto chunk_of = [](int row, int chunk) {
        return chunk ^ (((row & 3) << 1) | ((row >> 2) & 1));
    };
#pragma unroll
    for (int c = 0; c < D / 64; ++c) {
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x16& a = acc[2 * c + dt];
                uint2 w;
                w.x = pack_bf16(a[4 * r4] * f, a[4 * r4 + 1] * f);
                w.y = pack_bf16(a[4 * r4 + 2] * f, a[4 * r4 + 3] * f);
                *(uint2*)(lds + l32 * 128 + chunk_of(l32, 4 * dt + r4) * 16 + 8 * half) = w;
            }
        lane_exchange();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = 8 * j + (lane >> 3), pos = pos0 + t;
            const int64_t tok = (int64_t)(pos >> shift) * g.grid_w + (pos & (g.block_w - 1));
            *(uint4*)(block + tok * D + 64 * c + chunk_of(t, lane & 7) * 8) =
                *(const uint4*)(lds + 1024 * j + 16 * lane);
        }
        lane_exchange();
    }
}

// The same, added to what the rows hold together with extra * inv_b (extra: fp32, D
// channels).  32 channels at a time, which fp32 takes the same 4 KiB for.
template <int D>
__device__ __forceinline__ void add_rows(uint16_t* block, const Geom& g, int pos0,
                                         const f32x16 (&acc)[D / 32], float f, const float* extra,
                                         float inv_b, unsigned char* lds, int lane)
{
    const int l32 = lane & 31, half = lane >> 5, part = lane & 3;
    const int shift = __builtin_ctz((unsigned)g.block_w);
    auto chunk_of = [](int row, int chunk) {
        return chunk ^ (((row & 3) << 1) | ((row >> 2) & 1));
    };
    uint16_t* row[2];
    uint4 old[2][D / 32];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int pos = pos0 + 16 * j + (lane >> 2);
        row[j] = block + ((int64_t)(pos >> shift) * g.grid_w + (pos & (g.block_w - 1))) * D + 8 * part;
#pragma unroll
        for (int c = 0; c < D / 32; ++c) old[j][c] = *(const uint4*)(row[j] + 32 * c);
    }
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
            *(float4*)(lds + l32 * 128 + chunk_of(l32, 2 * r4 + half) * 16) =
                make_float4(acc[c][4 * r4] * f, acc[c][4 * r4 + 1] * f, acc[c][4 * r4 + 2] * f,
                            acc[c][4 * r4 + 3] * f);
        lane_exchange();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = 16 * j + (lane >> 2);
            const uint32_t o[4] = {old[j][c].x, old[j][c].y, old[j][c].z, old[j][c].w};
            uint32_t w[4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float4 v = *(const float4*)(lds + t * 128 + chunk_of(t, 2 * part + u) * 16);
                const float4 e = *(const float4*)(extra + 32 * c + 8 * part + 4 * u);
                const float x0 = v.x + (__uint_as_float(o[2 * u] << 16) + e.x * inv_b);
                const float x1 = v.y + (__uint_as_float(o[2 * u] & 0xffff0000u) + e.y * inv_b);
                const float x2 = v.z + (__uint_as_float(o[2 * u + 1] << 16) + e.z * inv_b);
                const float x3 = v.w + (__uint_as_float(o[2 * u + 1] & 0xffff0000u) + e.w * inv_b);
                w[2 * u] = pack_bf16(x0, x1);
                w[2 * u + 1] = pack_bf16(x2, x3);
            }
            *(uint4*)(row[j] + 32 * c) = make_uint4(w[0], w[1], w[2], w[3]);
        }
        lane_exchange();
    }
}

}  // namespace bsa
