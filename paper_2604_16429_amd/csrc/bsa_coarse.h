// The coarse-grained branch of the three-branch output for a group of query blocks
// (gfx950): a workgroup's work, shared by the kernel that does only this and by the
// one that ranks beside it.
#pragma once

#include "bsa_device.h"

namespace bsa {

constexpr float kCoarseLog2e = 1.4426950408889634f;
constexpr int kCoarseRows = 8;                      // most query blocks per workgroup
constexpr size_t kCoarseLdsBudget = 144 * 1024;

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    return v;
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}


// One workgroup of 256 threads handles G <= 8 consecutive query blocks of one
// (batch, head).
//   phase 1: thread t owns key block j = chunk*256 + t, holds kbar_j in
//            registers and scores it against the G pooled queries (scalar
//            operands); scaled scores (base-2 domain) land in LDS.
//   phase 2: one wavefront per query block: row maximum, weights
//            exp2(s - max) written back in place, 1 / row sum.
//   phase 3: thread = (channel quad, key partition): walks the pooled values
//            of its key partition (a row of vbar is read by D/4 adjacent
//            lanes, 16 bytes each) and accumulates weight * value for all G
//            rows in registers.
//   phase 4: the partitions' partial rows are summed, first inside each
//            wavefront (lanes with the same channel quad), then through LDS,
//            in fixed order, and scaled by 1 / row sum.
// LDS: G*m (scores) + 4*G*D (partials) + G floats.
template <int D>
__device__ __forceinline__ void coarse_block(const float* __restrict__ qbar,
                                             const float* __restrict__ kbar_il,
                                             const float* __restrict__ vbar,
                                             float* __restrict__ obar, const Geom& g, int G,
                                             uint32_t vblock)
{
    constexpr int CG = D / 4;                        // channel quads
    constexpr int JP = 256 / CG;                     // key partitions
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int m = g.n_blocks;
    float* red_s = (float*)smem;                     // [4 wavefronts][G][D]
    float* inv_s = red_s + 4 * G * D;                // [8]
    float* sc_s = inv_s + kCoarseRows;               // [G][m]

    const int groups = (m + G - 1) / G;
    const int64_t bh_idx = vblock / (uint32_t)groups;
    const int i0 = (int)(vblock - (uint32_t)bh_idx * (uint32_t)groups) * G;
    const int rows = min(G, m - i0);
    const int64_t kv = kv_slice_of(g, bh_idx);
    qbar += (bh_idx * m + i0) * D;
    vbar += kv * m * D;

    kbar_il += kv * m * D;                           // per slice [D/4][m][4]

    // ---- phase 1: scaled scores.  The pooled queries are wave-uniform (scalar
    // loads, scalar operands of the fma); the thread's pooled key comes from the
    // channel-interleaved copy (coalesced).
    const float c2 = g.scale * kCoarseLog2e;
    for (int j = threadIdx.x; j < m; j += blockDim.x) {
        float kr[D];
        const float4* ksrc = (const float4*)kbar_il + j;
#pragma unroll
        for (int d4 = 0; d4 < D / 4; ++d4) {
            const float4 t = ksrc[(int64_t)d4 * m];
            kr[4 * d4 + 0] = t.x; kr[4 * d4 + 1] = t.y;
            kr[4 * d4 + 2] = t.z; kr[4 * d4 + 3] = t.w;
        }
        for (int r = 0; r < rows; ++r) {
            const float* __restrict__ qrow = qbar + r * D;
            float acc = 0.0f;
#pragma unroll
            for (int d = 0; d < D; ++d) acc = fmaf(qrow[d], kr[d], acc);
            sc_s[r * m + j] = acc * c2;
        }
    }
    __syncthreads();

    // ---- phase 2: softmax weights per row, one wavefront each
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int r = wave; r < rows; r += 4) {
        float* row = sc_s + r * m;
        float mx = -INFINITY;
        for (int j = lane; j < m; j += 64) mx = fmaxf(mx, row[j]);
        mx = wave_max(mx);
        float sum = 0.0f;
        for (int j = lane; j < m; j += 64) {
            const float w = __builtin_amdgcn_exp2f(row[j] - mx);
            row[j] = w;
            sum += w;
        }
        sum = wave_sum(sum);
        if (lane == 0) inv_s[r] = 1.0f / sum;
    }
    __syncthreads();

    // ---- phase 3: weights times pooled values
    const int cg = threadIdx.x % CG, jp = threadIdx.x / CG;
    float4 acc[kCoarseRows];
#pragma unroll
    for (int r = 0; r < kCoarseRows; ++r) acc[r] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int j = jp; j < m; j += JP) {
        const float4 val = *(const float4*)(vbar + (int64_t)j * D + 4 * cg);
#pragma unroll
        for (int r = 0; r < kCoarseRows; ++r) {
            if (r < rows) {
                const float w = sc_s[r * m + j];
                acc[r].x = fmaf(w, val.x, acc[r].x);
                acc[r].y = fmaf(w, val.y, acc[r].y);
                acc[r].z = fmaf(w, val.z, acc[r].z);
                acc[r].w = fmaf(w, val.w, acc[r].w);
            }
        }
    }
    // ---- phase 4: the 64 / CG partitions of a wavefront hold the same channel
    // quad CG lanes apart: butterfly sums, then one partial row per wavefront
#pragma unroll
    for (int r = 0; r < kCoarseRows; ++r)
        for (int off = CG; off < 64; off <<= 1) {
            acc[r].x += __shfl_xor(acc[r].x, off);
            acc[r].y += __shfl_xor(acc[r].y, off);
            acc[r].z += __shfl_xor(acc[r].z, off);
            acc[r].w += __shfl_xor(acc[r].w, off);
        }
    if (lane < CG) {
#pragma unroll
        for (int r = 0; r < kCoarseRows; ++r)
            if (r < rows) *(float4*)(red_s + ((wave * G + r) * D) + 4 * cg) = acc[r];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < rows * D; e += blockDim.x) {
        const int r = e / D, d = e - r * D;
        float sum = 0.0f;
        for (int p = 0; p < 4; ++p) sum += red_s[(p * G + r) * D + d];
        obar[(bh_idx * m + i0 + r) * D + d] = sum * inv_s[r];
    }
}

inline size_t coarse_lds_bytes(int G, int m, int D)
{
    return ((size_t)4 * G * D + kCoarseRows + (size_t)G * m) * 4;
}

inline int coarse_group_size(int m, int D)
{
    for (int G = kCoarseRows; G >= 1; G >>= 1)
        if (coarse_lds_bytes(G, m, D) <= kCoarseLdsBudget) return G;
    return 0;
}

// Query blocks per workgroup: as many as fit, fewer when that would leave less than
// two workgroups per CU.
inline int coarse_group_for(int m, int D, int64_t BH)
{
    int G = coarse_group_size(m, D);
    while (G > 1 && BH * ((m + G - 1) / G) < 512) G >>= 1;
    return G;
}

}  // namespace bsa
