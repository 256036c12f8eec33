// The pieces of the paper's three-branch output that the single-softmax path
// does not already have (gfx950):
//
//   coarse_kernel        coarse-grained branch: for query block i the softmax
//                        over ALL m key blocks of qbar_i . kbar_j / sqrt(d_k)
//                        (block-level attention equation) applied to the
//                        mean-pooled values (coarse-grained output equation);
//                        one fp32 row [D] per query block.
//   combine_kernel       o = g_cg * o_cg(block of the token) + g_fg * o_fg +
//                        g_l * o_l with caller-supplied gate values
//                        (aggregation equation of the Native Sparse Attention
//                        subsection).  HBM-bound, one pass.
//
// The selection branch is the forward kernel in its list-only mode, the local branch
// the forward kernel run on "tile i and the other tiles of its large block" (Local
// Attention paragraph; the pooling launch writes those lists).
#include "bsa_coarse.h"
#include "bsa_device.h"
#include "bsa_launch.h"
#include "bsa_mfma_common.h"

namespace bsa {

template <int D>
__global__ __launch_bounds__(256) void coarse_kernel(const float* __restrict__ qbar,
                                                     const float* __restrict__ kbar_il,
                                                     const float* __restrict__ vbar,
                                                     float* __restrict__ obar, Geom g, int G)
{
    coarse_block<D>(qbar, kbar_il, vbar, obar, g, G, blockIdx.x);
}

template <int D>
static hipError_t launch_coarse_t(const float* qbar, const float* kbar_il, const float* vbar,
                                  float* obar, const Geom& g, int64_t BH, hipStream_t stream)
{
    const int G = coarse_group_for(g.n_blocks, D, BH);
    if (G == 0) return hipErrorInvalidValue;
    // the attribute is per device; setting it twice (two host threads racing) is harmless
    static bool attr_set[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!attr_set[dev]) {
        hipError_t e = hipFuncSetAttribute((const void*)coarse_kernel<D>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kCoarseLdsBudget);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    dim3 grid((unsigned)(BH * ((g.n_blocks + G - 1) / G)));
    hipLaunchKernelGGL((coarse_kernel<D>), grid, dim3(256), coarse_lds_bytes(G, g.n_blocks, D),
                       stream, qbar, kbar_il, vbar, obar, g, G);
    return hipGetLastError();
}

hipError_t launch_coarse(const float* qbar, const float* kbar_il, const float* vbar, float* obar,
                         const Geom& g, int D, int64_t BH, hipStream_t stream)
{
    switch (D) {
    case 32: return launch_coarse_t<32>(qbar, kbar_il, vbar, obar, g, BH, stream);
    case 64: return launch_coarse_t<64>(qbar, kbar_il, vbar, obar, g, BH, stream);
    case 128: return launch_coarse_t<128>(qbar, kbar_il, vbar, obar, g, BH, stream);
    }
    return hipErrorInvalidValue;
}

// One thread per VEC consecutive channels of one token.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void combine_kernel(const float* __restrict__ obar,
                                                      const T* __restrict__ o_fg,
                                                      const T* __restrict__ o_l,
                                                      const float* __restrict__ gates,
                                                      T* __restrict__ out, Geom g, int D,
                                                      int64_t total)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int per_row = D / VEC;
    const int64_t row = e / per_row;                 // bh * N + token
    const int ch = (int)(e - row * per_row) * VEC;
    const int64_t bh = row / g.n_tokens;
    const int64_t tok = row - bh * g.n_tokens;
    const int gr = (int)(tok / g.grid_w), gc = (int)(tok - (int64_t)gr * g.grid_w);
    const int beta = (gr / g.block_h) * g.blocks_per_row + gc / g.block_w;
    const float g_cg = gates[row * 3 + 0], g_fg = gates[row * 3 + 1], g_l = gates[row * 3 + 2];
    const float* ob = obar + (bh * g.n_blocks + beta) * D + ch;
#pragma unroll
    for (int v = 0; v < VEC; v += 4) {
        const float4 a = *(const float4*)(ob + v);
        const float4 f = load4(o_fg + row * D + ch + v);
        const float4 l = load4(o_l + row * D + ch + v);
        float4 o;
        o.x = fmaf(g_cg, a.x, fmaf(g_fg, f.x, g_l * l.x));
        o.y = fmaf(g_cg, a.y, fmaf(g_fg, f.y, g_l * l.y));
        o.z = fmaf(g_cg, a.z, fmaf(g_fg, f.z, g_l * l.z));
        o.w = fmaf(g_cg, a.w, fmaf(g_fg, f.w, g_l * l.w));
        store4(out + row * D + ch + v, o);
    }
}

hipError_t launch_combine(bool is_bf16, const float* obar, const void* o_fg, const void* o_l,
                          const float* gates, void* out, const Geom& g, int D, int64_t BH,
                          hipStream_t stream)
{
    if (is_bf16) {
        const int64_t total = BH * g.n_tokens * (D / 8);
        hipLaunchKernelGGL((combine_kernel<uint16_t, 8>), dim3((unsigned)((total + 255) / 256)),
                           dim3(256), 0, stream, obar, (const uint16_t*)o_fg,
                           (const uint16_t*)o_l, gates, (uint16_t*)out, g, D, total);
    } else {
        const int64_t total = BH * g.n_tokens * (D / 4);
        hipLaunchKernelGGL((combine_kernel<float, 4>), dim3((unsigned)((total + 255) / 256)),
                           dim3(256), 0, stream, obar, (const float*)o_fg, (const float*)o_l,
                           gates, (float*)out, g, D, total);
    }
    return hipGetLastError();
}


// ---------------------------------------------------------------------------
// Backward of the three-branch output (selection held fixed).
//   branch_grads_kernel  dO_fg = g_fg * dO and dO_l = g_l * dO (what the
//                        attention backward kernels of the two branches take
//                        as upstream gradient), delta and the base-2 log-sum-exps of
//                        both branches, the gate gradients dg_b = dO . o_b per
//                        token, and d(coarse row of block i) = sum over the
//                        tokens l of the block of g_cg(l) * dO_l, fp32 [B*h, m, D].
//   coarse_bwd_rows_kernel  per query block: block attention a_i, da_ij =
//                        dobar_i . vbar_j, ds_ij = a_ij (da_ij - sum_j a_ij
//                        da_ij); writes a and ds and dqbar_i = scale * sum_j
//                        ds_ij kbar_j.
//   coarse_bwd_cols_kernel  per key block and key/value slice: dvbar_j =
//                        sum_i a_ij dobar_i and dkbar_j = scale * sum_i ds_ij
//                        qbar_i.
// The two kernels alternate over chunks of R query blocks, so that a and ds
// are fp32 [B*h, R, m] with R chosen by the caller's scratch size, not
// [B*h, m, m]: the column kernel carries its sums from chunk to chunk in
// dkbar / dvbar (unscaled until the last chunk).  Summation order: chunks
// ascending, inside a chunk the query heads of the group ascending, inside a
// head the query blocks ascending.
// The pooled gradients reach the tokens in the local branch's attention
// backward, whose stores add (pooled gradient of the token's block) / b: the
// mean pooling hands every token of a block the same share.
// ---------------------------------------------------------------------------
// 16 bytes as fp32 channels
template <typename W> __device__ __forceinline__ void widen(const W& w, float (&x)[8])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[2 * e] = __uint_as_float(w[e] << 16);
        x[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
}
template <typename W> __device__ __forceinline__ void widen(const W& w, float (&x)[4])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(w[e]);
}

// x times f in the stored type.
template <typename W> __device__ __forceinline__ void narrow(const float (&x)[8], float f, W& w)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = pack_bf16(f * x[2 * e], f * x[2 * e + 1]);
}
template <typename W> __device__ __forceinline__ void narrow(const float (&x)[4], float f, W& w)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = __float_as_uint(f * x[e]);
}

// The value of lane t of this lane's quad.
__device__ __forceinline__ float quad_lane(float x, int t)
{
    const int i = __float_as_int(x);
    return __int_as_float(t == 0   ? __builtin_amdgcn_update_dpp(0, i, 0x00, 0xf, 0xf, false)
                          : t == 1 ? __builtin_amdgcn_update_dpp(0, i, 0x55, 0xf, 0xf, false)
                          : t == 2 ? __builtin_amdgcn_update_dpp(0, i, 0xaa, 0xf, 0xf, false)
                                   : __builtin_amdgcn_update_dpp(0, i, 0xff, 0xf, 0xf, false));
}

// One pass over dO and the two branch outputs.  A group of D/VEC adjacent lanes walks
// the tokens of a quarter of a tile in in-tile order, VEC channels (16 bytes) per
// lane: the dot products are summed inside the group, the gated sum of dO stays in
// the lane's registers and the four quarters of a tile, which are neighbours in a
// workgroup, are added through LDS in order.  delta of a branch is taken from the
// upstream gradient as it is stored, i.e. rounded: the attention backward computes dP
// from the same values, and in dP - delta their rounding then cancels for the most
// part (gate times gate gradient, which needs no sum of its own, has no such luck).
// One launch where there were four (gradients, gated sums, delta of each branch).
template <typename T, int D>
__global__ __launch_bounds__(256) void branch_grads_kernel(
    const float* __restrict__ obar, const T* __restrict__ o_fg, const T* __restrict__ o_l,
    const float* __restrict__ lse_fg, const float* __restrict__ lse_l,
    const float* __restrict__ gates, const T* __restrict__ dout, T* __restrict__ do_fg,
    T* __restrict__ do_l, float* __restrict__ dgates, float* __restrict__ dobar,
    float* __restrict__ delta_fg, float* __restrict__ delta_l, float* __restrict__ lse2_fg,
    float* __restrict__ lse2_l, Geom g, int64_t tiles)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int VEC = 16 / (int)sizeof(T), LANES = D / VEC;       // 4 to 32 lanes per token
    constexpr int PARTS = 4, TILES = 256 / (LANES * PARTS);         // tiles per workgroup
    constexpr int BATCH = 4;                                        // tokens in flight
    __shared__ float sum_s[PARTS][TILES][D];
    const int mine = threadIdx.x & 3;
    const int lane = (int)threadIdx.x % LANES, part = ((int)threadIdx.x / LANES) % PARTS;
    const int slot = (int)threadIdx.x / (LANES * PARTS);
    int64_t tile = (int64_t)blockIdx.x * TILES + slot;              // bh * m + beta
    const bool valid = tile < tiles;
    if (!valid) tile = tiles - 1;                                   // keep the lane groups whole
    const int64_t bh = tile / g.n_blocks;
    const int beta = (int)(tile - bh * g.n_blocks);
    const int ch = lane * VEC;
    const int b = g.block_tokens;
    float ob[VEC], acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; v += 4) {
        const float4 t = *(const float4*)(obar + tile * D + ch + v);
        ob[v] = t.x; ob[v + 1] = t.y; ob[v + 2] = t.z; ob[v + 3] = t.w;
        acc[v] = acc[v + 1] = acc[v + 2] = acc[v + 3] = 0.0f;
    }
    const int tau_end = b * (part + 1) / PARTS;
    int tau = b * part / PARTS, col = tau % g.block_w;
    int64_t row = bh * g.n_tokens + token_of(g, beta, tau);         // of the next token
    const int row_jump = g.grid_w - g.block_w;
    while (tau < tau_end) {
        const int count = min(BATCH, tau_end - tau);
        int64_t rows[BATCH];
        u32x4 w_up[BATCH], w_f[BATCH], w_l[BATCH];
#pragma unroll
        for (int t = 0; t < BATCH; ++t) {
            rows[t] = row;
            // (past the part's last token: that token again)
            if (t + 1 < count || (t + 1 == count && tau + BATCH < tau_end)) {
                ++row;
                if (++col == g.block_w) { col = 0; row += row_jump; }
            }
            w_up[t] = *(const u32x4*)(dout + rows[t] * D + ch);
            w_f[t] = *(const u32x4*)(o_fg + rows[t] * D + ch);
            w_l[t] = *(const u32x4*)(o_l + rows[t] * D + ch);
        }
        // scalars of a token: the lane whose number is t modulo 4 reads and writes
        // those of token t, so that a wavefront's accesses cover runs of tokens; the
        // others get them inside their quad
        const int64_t my_row = mine == 0 ? rows[0] : mine == 1 ? rows[1]
                               : mine == 2 ? rows[2] : rows[3];
        float my_gate[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) my_gate[x] = gates[my_row * 3 + x];
        const float my_fg = lse_fg[my_row], my_l = lse_l[my_row];
        float my_cg = 0.0f, my_dfg = 0.0f, my_dl = 0.0f, my_efg = 0.0f, my_el = 0.0f;
#pragma unroll
        for (int t = 0; t < BATCH; ++t) {
            const bool live = t < count;
            const float g_cg = quad_lane(my_gate[0], t), g_fg = quad_lane(my_gate[1], t),
                        g_l = quad_lane(my_gate[2], t);
            float up[VEC], f[VEC], l[VEC];
            widen(w_up[t], up);
            widen(w_f[t], f);
            widen(w_l[t], l);
            u32x4 s_fg, s_l;
            narrow(up, g_fg, s_fg);
            narrow(up, g_l, s_l);
            float up_fg[VEC], up_l[VEC];                            // as they are stored
            widen(s_fg, up_fg);
            widen(s_l, up_l);
            float d_cg = 0.0f, d_fg = 0.0f, d_l = 0.0f, e_fg = 0.0f, e_l = 0.0f;
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                d_cg = fmaf(up[v], ob[v], d_cg);
                d_fg = fmaf(up[v], f[v], d_fg);
                d_l = fmaf(up[v], l[v], d_l);
                e_fg = fmaf(up_fg[v], f[v], e_fg);
                e_l = fmaf(up_l[v], l[v], e_l);
                if (live) acc[v] = fmaf(g_cg, up[v], acc[v]);
            }
            if (valid && live) {
                *(u32x4*)(do_fg + rows[t] * D + ch) = s_fg;
                *(u32x4*)(do_l + rows[t] * D + ch) = s_l;
            }
#pragma unroll
            for (int off = LANES >> 1; off >= 1; off >>= 1) {
                d_cg += __shfl_xor(d_cg, off);
                d_fg += __shfl_xor(d_fg, off);
                d_l += __shfl_xor(d_l, off);
                e_fg += __shfl_xor(e_fg, off);
                e_l += __shfl_xor(e_l, off);
            }
            my_efg = mine == t ? e_fg : my_efg;
            my_el = mine == t ? e_l : my_el;
            my_cg = mine == t ? d_cg : my_cg;
            my_dfg = mine == t ? d_fg : my_dfg;
            my_dl = mine == t ? d_l : my_dl;
        }
        if (valid && lane < count) {                                // lane < 4: mine == lane
            dgates[my_row * 3] = my_cg;
            dgates[my_row * 3 + 1] = my_dfg;
            dgates[my_row * 3 + 2] = my_dl;
            delta_fg[my_row] = my_efg;
            delta_l[my_row] = my_el;
            lse2_fg[my_row] = my_fg * kCoarseLog2e;
            lse2_l[my_row] = my_l * kCoarseLog2e;
        }
        tau += BATCH;
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) sum_s[part][slot][ch + v] = acc[v];
    __syncthreads();
    for (int e = threadIdx.x; e < TILES * D; e += 256) {
        const int t = e / D, d = e - t * D;
        const int64_t out_tile = (int64_t)blockIdx.x * TILES + t;
        if (out_tile < tiles)
            dobar[out_tile * D + d] =
                ((sum_s[0][t][d] + sum_s[1][t][d]) + sum_s[2][t][d]) + sum_s[3][t][d];
    }
}

// Same workgroup shape as coarse_kernel (G <= 8 query blocks of one slice).
// LDS: 4*G*D (partials) + 2*G*m (weights, ds) floats.
template <int D>
__global__ __launch_bounds__(256) void coarse_bwd_rows_kernel(
    const float* __restrict__ qbar, const float* __restrict__ kbar,
    const float* __restrict__ kbar_il, const float* __restrict__ vbar,
    const float* __restrict__ dobar, float* __restrict__ a_out, float* __restrict__ ds_out,
    float* __restrict__ dqbar, Geom g, int G, int R, int r0, int r1)
{
    // query blocks r0 .. r1-1 of every slice; a_out, ds_out: [B*h, R, m] with
    // R >= r1 - r0
    constexpr int CG = D / 4, JP = 256 / CG;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int m = g.n_blocks;
    float* red_s = (float*)smem;                     // [4 wavefronts][G][D]
    float* sc_s = red_s + 4 * G * D;                 // [G][m]: scores -> weights a
    float* da_s = sc_s + G * m;                      // [G][m]: da -> ds

    const int groups = (r1 - r0 + G - 1) / G;
    const int64_t bh_idx = blockIdx.x / groups;
    const int i0 = r0 + (int)(blockIdx.x - bh_idx * groups) * G;
    const int rows = min(G, r1 - i0);
    const int64_t kv = kv_slice_of(g, bh_idx);
    kbar += kv * m * D;
    vbar += kv * m * D;
    const int64_t row0 = bh_idx * m + i0;
    const int64_t out_row0 = bh_idx * R + (i0 - r0);    // row of a_out / ds_out
    kbar_il += kv * m * D;                           // per slice [D/4][m][4]

    // scores (base-2 domain) and da_ij = dobar_i . vbar_j; the rows of qbar and
    // dobar are wave-uniform (scalar loads, scalar operands of the fma)
    const float c2 = g.scale * kCoarseLog2e;
    for (int j = threadIdx.x; j < m; j += blockDim.x) {
        float kr[D];
        const float4* ksrc = (const float4*)kbar_il + j;
#pragma unroll
        for (int d4 = 0; d4 < D / 4; ++d4) {
            const float4 t = ksrc[(int64_t)d4 * m];
            kr[4 * d4 + 0] = t.x; kr[4 * d4 + 1] = t.y; kr[4 * d4 + 2] = t.z; kr[4 * d4 + 3] = t.w;
        }
        for (int r = 0; r < rows; ++r) {
            const float* __restrict__ qrow = qbar + (row0 + r) * D;
            float acc = 0.0f;
#pragma unroll
            for (int d = 0; d < D; ++d) acc = fmaf(qrow[d], kr[d], acc);
            sc_s[r * m + j] = acc * c2;
        }
#pragma unroll
        for (int d4 = 0; d4 < D / 4; ++d4) {
            const float4 t = *(const float4*)(vbar + (int64_t)j * D + 4 * d4);
            kr[4 * d4 + 0] = t.x; kr[4 * d4 + 1] = t.y; kr[4 * d4 + 2] = t.z; kr[4 * d4 + 3] = t.w;
        }
        for (int r = 0; r < rows; ++r) {
            const float* __restrict__ dorow = dobar + (row0 + r) * D;
            float acc = 0.0f;
#pragma unroll
            for (int d = 0; d < D; ++d) acc = fmaf(dorow[d], kr[d], acc);
            da_s[r * m + j] = acc;
        }
    }
    __syncthreads();

    // softmax weights and sum_j a_ij da_ij, one wavefront per row
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
        const float inv = 1.0f / wave_sum(sum);
        float dot = 0.0f;
        for (int j = lane; j < m; j += 64) {
            const float a = row[j] * inv;
            row[j] = a;
            dot = fmaf(a, da_s[r * m + j], dot);
        }
        dot = wave_sum(dot);
        // ds_ij, and both matrices to global memory for the column pass
        float* a_row = a_out + (out_row0 + r) * (int64_t)m;
        float* ds_row = ds_out + (out_row0 + r) * (int64_t)m;
        for (int j = lane; j < m; j += 64) {
            const float a = row[j];
            const float ds = a * (da_s[r * m + j] - dot);
            da_s[r * m + j] = ds;
            a_row[j] = a;
            ds_row[j] = ds;
        }
    }
    __syncthreads();

    // dqbar_i = scale * sum_j ds_ij kbar_j
    const int cg = threadIdx.x % CG, jp = threadIdx.x / CG;
    float4 acc[kCoarseRows];
#pragma unroll
    for (int r = 0; r < kCoarseRows; ++r) acc[r] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int j = jp; j < m; j += JP) {
        const float4 val = *(const float4*)(kbar + (int64_t)j * D + 4 * cg);
#pragma unroll
        for (int r = 0; r < kCoarseRows; ++r) {
            if (r < rows) {
                const float w = da_s[r * m + j];
                acc[r].x = fmaf(w, val.x, acc[r].x);
                acc[r].y = fmaf(w, val.y, acc[r].y);
                acc[r].z = fmaf(w, val.z, acc[r].z);
                acc[r].w = fmaf(w, val.w, acc[r].w);
            }
        }
    }
    // the partitions of a wavefront hold the same channel quad CG lanes apart
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
        dqbar[(row0 + r) * D + d] = sum * g.scale;
    }
}

static size_t coarse_bwd_lds_bytes(int G, int m, int D)
{
    return ((size_t)4 * G * D + (size_t)2 * G * m) * 4;
}

int coarse_bwd_group_size(int m, int D)
{
    for (int G = kCoarseRows; G >= 1; G >>= 1)
        if (coarse_bwd_lds_bytes(G, m, D) <= kCoarseLdsBudget) return G;
    return 0;
}

// The two column sums are matrix products, dvbar = a^T dobar and dkbar = ds^T qbar,
// with the query blocks (of all heads of a group) as the contraction: fp32 matrix
// instructions (v_mfma_f32_32x32x2_f32), a wavefront per 32 key blocks x 32
// channels of one of them.  Both operands come straight from memory, two query
// blocks per instruction (lane half h: block i + h), consecutive lanes reading
// consecutive addresses; UNROLL instructions' operands are in flight.  Query blocks
// ascend, heads of the group ascending outside: a fixed order.
// The sums start from what dkbar / dvbar hold unless r0 == 0 and are scaled only
// when r1 == m, so a sequence of calls over ascending chunks adds every term once.
// (One lane per key block with the rows as scalar operands, as before, was a chain of
// m * heads-per-group scalar-load latencies on a few wavefronts: stage 2 at batch 8
// 381 -> 28 us.)
template <int D>
__global__ __launch_bounds__(256) void coarse_bwd_cols_kernel(
    const float* __restrict__ qbar, const float* __restrict__ dobar,
    const float* __restrict__ a_in, const float* __restrict__ ds_in, float* __restrict__ dkbar,
    float* __restrict__ dvbar, Geom g, int64_t waves, int R, int r0, int r1)
{
    constexpr int DT = D / 32, UNROLL = 8;
    const int m = g.n_blocks;
    const int j_tiles = (m + 31) / 32;
    const int64_t wave_id =
        (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (wave_id >= waves) return;                     // whole wavefront; no barriers below
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    // wave_id = ((slice * j_tiles + j tile) * DT + channel tile) * 2 + (0: values, 1: keys)
    const bool keys = (wave_id & 1) != 0;
    const int64_t rest = wave_id >> 1;
    const int dt = (int)(rest % DT);
    const int64_t kv = rest / DT / j_tiles;
    const int j0 = (int)(rest / DT - kv * j_tiles) * 32;
    const int64_t kv_heads = g.heads / g.kv_group;
    const int64_t bh_first = (kv / kv_heads) * g.heads + (kv % kv_heads) * g.kv_group;
    const int jc = j0 + l32 < m ? j0 + l32 : m - 1;   // an idle column repeats the last one
    float* out = (keys ? dkbar : dvbar) + kv * m * D + 32 * dt + l32;

    // accumulator register r: key block j0 + 8 (r/4) + 4 half + r%4, channel 32 dt + l32
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int j = j0 + 8 * (r >> 2) + 4 * half + (r & 3);
        acc[r] = r0 > 0 && j < m ? out[(int64_t)j * D] : 0.0f;
    }
    for (int gq = 0; gq < g.kv_group; ++gq) {
        const int64_t bh = bh_first + gq;
        const float* w_col = (keys ? ds_in : a_in) + bh * R * (int64_t)m + jc;
        const float* rows = (keys ? qbar : dobar) + bh * m * D + 32 * dt + l32;
        for (int i0 = r0; i0 < r1; i0 += 2 * UNROLL) {
            float w[UNROLL], x[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int i = i0 + 2 * u + half;
                const bool in = i < r1;
                w[u] = in ? w_col[(int64_t)(i - r0) * m] : 0.0f;
                x[u] = in ? rows[(int64_t)i * D] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[u], x[u], acc, 0, 0, 0);
        }
    }
    const float f = keys && r1 == m ? g.scale : 1.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int j = j0 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (j < m) out[(int64_t)j * D] = acc[r] * f;
    }
}

template <typename T, int D>
static hipError_t launch_branch_grads_t(const BranchGrads& x, const Geom& g, int64_t BH,
                                        hipStream_t stream)
{
    constexpr int TILES = 256 / (D * (int)sizeof(T) / 16 * 4);
    const int64_t m = g.n_blocks;
    return launch_slices(BH, 256 * (m / TILES + 1), [&](int64_t first, int64_t slices) {
        const int64_t tiles = slices * m, row = first * g.n_tokens, at = row * D, pooled = first * m * D;
        branch_grads_kernel<T, D><<<dim3((unsigned)((tiles + TILES - 1) / TILES)), dim3(256), 0,
                                    stream>>>(
            x.obar + pooled, (const T*)x.o_fg + at, (const T*)x.o_l + at, x.lse_fg + row,
            x.lse_l + row, x.gates + 3 * row, (const T*)x.dout + at, (T*)x.do_fg + at,
            (T*)x.do_l + at, x.dgates + 3 * row, x.dobar + pooled, x.delta_fg + row, x.delta_l + row,
            x.lse2_fg + row, x.lse2_l + row, g, tiles);
        return hipGetLastError();
    });
}

hipError_t launch_branch_grads(bool is_bf16, const BranchGrads& x, const Geom& g, int D, int64_t BH,
                               hipStream_t stream)
{
#define BSA_CASE(DD)                                                                  \
    case DD:                                                                          \
        return is_bf16 ? launch_branch_grads_t<uint16_t, DD>(x, g, BH, stream)        \
                       : launch_branch_grads_t<float, DD>(x, g, BH, stream);
    switch (D) {
        BSA_CASE(32)
        BSA_CASE(64)
        BSA_CASE(128)
    }
#undef BSA_CASE
    return hipErrorInvalidValue;
}

template <int D>
static hipError_t launch_coarse_bwd_t(const float* qbar, const float* kbar, const float* kbar_il,
                                      const float* vbar, const float* dobar, float* a_mat, float* ds_mat,
                                      float* dqbar, float* dkbar, float* dvbar, const Geom& g,
                                      int64_t BH, int chunk_rows, hipStream_t stream)
{
    const int G = coarse_bwd_group_size(g.n_blocks, D);
    if (G == 0) return hipErrorInvalidValue;
    static bool attr_set[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!attr_set[dev]) {
        hipError_t e = hipFuncSetAttribute((const void*)coarse_bwd_rows_kernel<D>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kCoarseLdsBudget);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    const int m = g.n_blocks;
    const int R = chunk_rows;
    if (R < 1) return hipErrorInvalidValue;
    const int64_t BKV = BH / g.kv_group;
    const int64_t waves = (int64_t)((m + 31) / 32) * (D / 32) * 2;    // per key/value slice
    for (int r0 = 0; r0 < m; r0 += R) {
        const int r1 = r0 + R < m ? r0 + R : m;
        hipLaunchKernelGGL((coarse_bwd_rows_kernel<D>),
                           dim3((unsigned)(BH * ((r1 - r0 + G - 1) / G))), dim3(256),
                           coarse_bwd_lds_bytes(G, m, D), stream, qbar, kbar, kbar_il, vbar, dobar,
                           a_mat, ds_mat, dqbar, g, G, R, r0, r1);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = launch_slices(BKV, 64 * waves + 256, [&](int64_t first, int64_t slices) {
            const int64_t q_rows = first * g.kv_group * m * D, mat = first * g.kv_group * R * m;
            coarse_bwd_cols_kernel<D><<<dim3((unsigned)((slices * waves + 3) / 4)), dim3(256), 0,
                                        stream>>>(
                qbar + q_rows, dobar + q_rows, a_mat + mat, ds_mat + mat, dkbar + first * m * D,
                dvbar + first * m * D, g, slices * waves, R, r0, r1);
            return hipGetLastError();
        });
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_coarse_bwd(const float* qbar, const float* kbar, const float* kbar_il,
                             const float* vbar, const float* dobar, float* a_mat, float* ds_mat, float* dqbar,
                             float* dkbar, float* dvbar, const Geom& g, int D, int64_t BH,
                             int chunk_rows, hipStream_t stream)
{
    switch (D) {
    case 32: return launch_coarse_bwd_t<32>(qbar, kbar, kbar_il, vbar, dobar, a_mat, ds_mat, dqbar, dkbar, dvbar, g, BH, chunk_rows, stream);
    case 64: return launch_coarse_bwd_t<64>(qbar, kbar, kbar_il, vbar, dobar, a_mat, ds_mat, dqbar, dkbar, dvbar, g, BH, chunk_rows, stream);
    case 128: return launch_coarse_bwd_t<128>(qbar, kbar, kbar_il, vbar, dobar, a_mat, ds_mat, dqbar, dkbar, dvbar, g, BH, chunk_rows, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace bsa
