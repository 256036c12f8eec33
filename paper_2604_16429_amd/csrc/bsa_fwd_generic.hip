// Block-sparse attention forward for every shape the specialised kernels do not
// cover, on the gfx950 matrix cores: fp32 and bf16, head dim 32, 64 or 128, any
// tile of up to 1024 tokens.
//
// Every token of query block i attends, in one softmax, to the tokens of block
// i and of its n selected blocks (fine-grained attention equation plus the
// local block).  A wavefront owns 32 query rows; a workgroup of up to 8
// wavefronts owns up to 256 rows of one query block, whose wavefronts attend to
// the same keys.  The attended keys are walked as one flat sequence
// (bsa_flat_rows.h) in tiles of 64 (bf16) or 32 (fp32) keys that the workgroup
// shares through LDS: gathered with direct-to-LDS loads, double buffered, one
// barrier per tile.
//
// Transposed products as in the specialised kernels: S^T = K Q^T and
// O^T = V^T P^T with 32x32 accumulators, so that a lane holds one query column,
// the softmax reductions are in-register, and the S^T accumulator registers are
// the B operand of the second product.
//   fp32: v_mfma_f32_32x32x2_f32, i.e. fp32 products and sums throughout.  Lane
//         half h supplies channels 8 j + 4 h + 0..3 of its row, so a 16-byte
//         read feeds four instructions; accumulator register r is, as it is, the
//         B operand of the keys 8 (r/4) + r%4 (+ 4 for the upper half).
//   bf16: v_mfma_f32_32x32x16_bf16.  The weights enter the second product as two
//         bf16 terms (16 significant bits): these shapes have always had their
//         weights multiplied in fp32, and keep that precision.
// Measured against the vector-ALU kernel that it replaces (one lane per query
// row, keys broadcast from LDS), select + forward: 131,072 tokens, 16 heads, head
// dim 32, bf16, 17 blocks of 128: 9.87 -> 1.39 ms; the 32 x 64 grid in fp32: 120
// -> 37 us.
// Softmax without a row maximum per tile: weights are taken against a reference
// that only moves when a row sum of a tile leaves the safe range.
#include "bsa_device.h"
#include "bsa_flat_rows.h"
#include "bsa_launch.h"
#include "bsa_mfma_common.h"

namespace bsa {

namespace {

__device__ __forceinline__ f32x16 zero_tile()
{
    const f32x16 z = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f,
                      0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    return z;
}

// S^T tile of 32 keys x 32 queries.  qf: this lane's query row (bf16: B operands
// of the 16-channel steps; fp32: the channels 8 j + 4 half + 0..3).
template <int D>
__device__ __forceinline__ f32x16 score_tile(const unsigned char* k_rows, const bf16x8 (&qf)[D / 16],
                                             int l32, int half)
{
    using Tile = FlatTile<uint16_t, D>;
    f32x16 s = zero_tile();
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        const bf16x8 kf = *(const bf16x8*)(k_rows + l32 * Tile::ROW_BYTES +
                                           Tile::swz(l32, 2 * ks + half) * 16);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s, 0, 0, 0);
    }
    return s;
}
template <int D>
__device__ __forceinline__ f32x16 score_tile(const unsigned char* k_rows, const float4 (&qf)[D / 8],
                                             int l32, int half)
{
    using Tile = FlatTile<float, D>;
    f32x16 s = zero_tile();
#pragma unroll
    for (int j = 0; j < D / 8; ++j) {
        const float4 kf = *(const float4*)(k_rows + l32 * Tile::ROW_BYTES +
                                           Tile::swz(l32, 2 * j + half) * 16);
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.x, qf[j].x, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.y, qf[j].y, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.z, qf[j].z, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf.w, qf[j].w, s, 0, 0, 0);
    }
    return s;
}

// O^T += V^T P^T for 32 keys; p: the weights in the accumulator layout.
template <int D>
__device__ __forceinline__ void value_tile(const uint16_t*, const unsigned char* v_rows,
                                           const f32x16& p, f32x16 (&oacc)[D / 32], int lane)
{
    using Tile = FlatTile<uint16_t, D>;
    const int s16 = lane & 15, gq = lane >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            split_bf16(p[8 * h + 2 * e], p[8 * h + 2 * e + 1], hi[e], lo[e]);
        const bf16x8 p_hi = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
        const bf16x8 p_lo = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
            // transposing read: source lane s of 16-lane group gq supplies 8 bytes
            // of V[16 h + 8 rd + 4 (gq/2) + s/4][32 dt + 16 (gq%2) + 4 (s%4)]
            const int col = 16 * (gq & 1) + 4 * (s16 & 3) + 32 * dt;
            bf16x4 part[2];
#pragma unroll
            for (int rd = 0; rd < 2; ++rd) {
                const int row = 16 * h + 8 * rd + 4 * (gq >> 1) + (s16 >> 2);
                const unsigned char* src = v_rows + row * Tile::ROW_BYTES +
                                           Tile::swz(row, col >> 3) * 16 + (col & 7) * 2;
                part[rd] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, src));
            }
            const bf16x8 vf = __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p_hi, oacc[dt], 0, 0, 0);
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p_lo, oacc[dt], 0, 0, 0);
        }
    }
}
template <int D>
__device__ __forceinline__ void value_tile(const float*, const unsigned char* v_rows,
                                           const f32x16& p, f32x16 (&oacc)[D / 32], int lane)
{
    using Tile = FlatTile<float, D>;
    const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * half + (r & 3);
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
            const int chunk = 8 * dt + (l32 >> 2);
            const float v = *(const float*)(v_rows + row * Tile::ROW_BYTES +
                                            Tile::swz(row, chunk) * 16 + (l32 & 3) * 4);
            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(v, p[r], oacc[dt], 0, 0, 0);
        }
    }
}

__device__ __forceinline__ void load_query(const uint16_t* row, bf16x8& f, int step, int half)
{
    f = *(const bf16x8*)(row + 16 * step + 8 * half);
}
__device__ __forceinline__ void load_query(const float* row, float4& f, int step, int half)
{
    f = *(const float4*)(row + 8 * step + 4 * half);
}

template <typename T, int D> struct QueryFrag;
template <int D> struct QueryFrag<uint16_t, D> { typedef bf16x8 type; static constexpr int N = D / 16; };
template <int D> struct QueryFrag<float, D> { typedef float4 type; static constexpr int N = D / 8; };

}  // namespace

// NL: wavefronts that issue the gathers (1, 2 or 4; the workgroup has at least
// that many, up to 8).  row_chunks workgroups share a query block's rows,
// chunk_rows each.
template <typename T, int D, int NL>
__global__ __launch_bounds__(NL == 4 ? 512 : NL == 2 ? 192 : 64, NL == 1 || (NL == 2 && D == 128) ? 1 : D == 32 ? 4 : 2)
void fwd_generic_kernel(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                        const int32_t* __restrict__ sel_idx, T* __restrict__ out,
                        float* __restrict__ lse, Geom g, uint32_t n_units, int row_chunks,
                        int chunk_rows)
{
    using Tile = FlatTile<T, D>;
    constexpr int KT = Tile::KT, MINE = Tile::SLABS / NL;
    static_assert(Tile::SLABS % NL == 0, "slabs split evenly between the loading wavefronts");
    __shared__ __attribute__((aligned(1024))) unsigned char k_lds[2][Tile::TILE_BYTES];
    __shared__ __attribute__((aligned(1024))) unsigned char v_lds[2][Tile::TILE_BYTES];
    extern __shared__ __attribute__((aligned(16))) uint32_t tables_s[];
    uint32_t* pos_s = tables_s;                        // [b]
    uint32_t* first_s = tables_s + g.block_tokens;     // [min(listed blocks, kListTable)]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int b = g.block_tokens;

    int item;
    int64_t bh_idx;
    map_workgroup(g, blockIdx.x, (uint32_t)(g.n_blocks * row_chunks), n_units, bh_idx, item);
    const int i = item / row_chunks;
    const int row0 = (item - i * row_chunks) * chunk_rows;
    const int64_t base = bh_idx * g.n_tokens * D;
    const int64_t kv_base = kv_slice_of(g, bh_idx) * g.n_tokens * D;
    // The attended blocks: block i itself followed by its selected blocks, or,
    // when the selection branch runs on its own, exactly the listed blocks.
    const int list_only = g.list_only;
    const int32_t* sel_row = sel_idx + (bh_idx * g.n_blocks + i) * g.n_select + list_only;
    const int first = list_only ? sel_row[-1] : i;
    const int n = g.n_select - list_only;        // blocks after the first

    // Tables.  Up to 63 listed blocks are visited in ascending order (query blocks
    // that run together then sweep the slice's K/V in the same direction).
    fill_position_table(g, pos_s);
    if (n < 64) {
        if (wave == 0) {
            const int mine = lane < n ? sel_row[lane] : 0x7fffffff;
            int rank = 1;
            for (int t = 0; t < n; ++t)
                rank += __builtin_amdgcn_readlane(mine, t) < mine ? 1 : 0;
            if (lane < n) first_s[rank] = block_first_token(g, mine);
            if (lane == 0) first_s[0] = block_first_token(g, first);
        }
    } else {
        for (int t = threadIdx.x; t <= n && t < kListTable; t += blockDim.x)
            first_s[t] = block_first_token(g, t == 0 ? first : sel_row[t - 1]);
    }

    // this wavefront's 32 query rows
    const int tau_q = row0 + 32 * wave + l32;
    const bool valid = tau_q < min(b, row0 + chunk_rows);
    int64_t q_tok;
    typename QueryFrag<T, D>::type qf[QueryFrag<T, D>::N];
    {
        const int t = valid ? tau_q : 0;
        const int rr = t / g.block_w;
        q_tok = (int64_t)block_first_token(g, i) + (int64_t)rr * g.grid_w + (t - rr * g.block_w);
#pragma unroll
        for (int s = 0; s < QueryFrag<T, D>::N; ++s)
            load_query(q + base + q_tok * D, qf[s], s, half);
    }
    __syncthreads();

    // this lane's rows of a tile: row RPS * slab + lane / LPR of slab wave + NL j
    const int total = (n + 1) * b;                   // attended keys
    const int tiles = (total + KT - 1) / KT;
    const int step_q = KT / b, step_r = KT - step_q * b;
    FlatRow at[MINE];
    uint32_t chunk_off[MINE];
#pragma unroll
    for (int j = 0; j < MINE; ++j) {
        const int row = Tile::RPS * (wave + NL * j) + lane / Tile::LPR;
        at[j].start(row, b);
        chunk_off[j] = (uint32_t)Tile::swz(row, lane % Tile::LPR) * 16u;
    }
    const unsigned char* kb = (const unsigned char*)(k + kv_base);
    const unsigned char* vb = (const unsigned char*)(v + kv_base);
    const uint32_t k_dst = lds_address(k_lds), v_dst = lds_address(v_lds);
    // gathers the next tile (rows past the end repeat the last row; they carry no
    // weight) and moves on
    auto gather_next = [&](int buf) {
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const bool past = at[j].blk > n;
            const int blk = past ? n : at[j].blk, tau = past ? b - 1 : at[j].tau;
            const uint32_t org = blk < kListTable ? first_s[blk]
                                                  : block_first_token(g, sel_row[blk - 1]);
            const uint64_t off = (uint64_t)(org + pos_s[tau]) * Tile::ROW_BYTES + chunk_off[j];
            const uint32_t dst = (uint32_t)buf * Tile::TILE_BYTES + (uint32_t)(wave + NL * j) * 1024u;
            load_lds_16_at(kb + off, k_dst + dst);
            load_lds_16_at(vb + off, v_dst + dst);
            at[j].advance(step_q, step_r, b);
        }
    };
    if (wave < NL) gather_next(0);

    const float c2 = g.scale * 1.4426950408889634f;
    f32x16 oacc[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) oacc[dt] = zero_tile();
    float m_ref = -INFINITY, l_run = 0.0f;

    for (int c = 0; c < tiles; ++c) {
        // tile c has landed and everyone is done with the other buffer
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (wave < NL && c + 1 < tiles) gather_next((c + 1) & 1);
        const unsigned char* kt = k_lds[c & 1];
        const unsigned char* vt = v_lds[c & 1];
#pragma unroll
        for (int hh = 0; hh < KT / 32; ++hh) {
            f32x16 s = score_tile<D>(kt + 32 * hh * Tile::ROW_BYTES, qf, l32, half);
            const int left = total - (KT * c + 32 * hh);     // keys from this half tile on
            if (left < 32) {
                if (left <= 0) break;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + 4 * half + (r & 3) >= left) s[r] = -INFINITY;
            }
            f32x16 p;
            float rs0 = 0.0f, rs1 = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -m_ref));
                p[r + 1] = __builtin_amdgcn_exp2f(fmaf(s[r + 1], c2, -m_ref));
                rs0 += p[r];
                rs1 += p[r + 1];
            }
            float rs = rs0 + rs1;
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(rs <= kSumLimit)) != 0, 0)) {
                // new reference from the row maxima; rescale what is there
                float mx = s[0];
#pragma unroll
                for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
                mx = fmaxf(mx, swap32(mx));
                const float m_new = fmaxf(m_ref, mx * c2);
                const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);
                m_ref = m_new;
                l_run *= alpha;
#pragma unroll
                for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
                rs = 0.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -m_new));
                    rs += p[r];
                }
            }
            l_run += rs;
            value_tile<D>((const T*)nullptr, vt + 32 * hh * Tile::ROW_BYTES, p, oacc, lane);
        }
    }

    const float l_tot = l_run + swap32(l_run);
    if (valid) {
        const float inv_l = 1.0f / l_tot;
        T* orow = out + base + q_tok * D;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                store4(orow + 32 * dt + 8 * r4 + 4 * half,
                       make_float4(oacc[dt][4 * r4] * inv_l, oacc[dt][4 * r4 + 1] * inv_l,
                                   oacc[dt][4 * r4 + 2] * inv_l, oacc[dt][4 * r4 + 3] * inv_l));
        if (lse && half == 0)
            lse[bh_idx * g.n_tokens + q_tok] =
                (m_ref + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f;
    }
}

template <typename T, int D>
static hipError_t launch_t(const void* q, const void* k, const void* v, const int32_t* sel_idx,
                           void* out, float* lse, const Geom& g, int64_t BH, hipStream_t stream)
{
    // rows of a query block: as few workgroups of at most 8 wavefronts as hold
    // them, as even as possible in units of 32 rows
    const int row_tiles = (g.block_tokens + 31) / 32;
    const int row_chunks = (row_tiles + 7) / 8;
    const int nw = (row_tiles + row_chunks - 1) / row_chunks;
    if (BH * g.n_blocks * row_chunks >= (int64_t)1 << 31) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(BH * g.n_blocks * row_chunks)), block(64 * nw);
    auto kernel = nw >= 4 ? fwd_generic_kernel<T, D, 4>
                  : nw >= 2 ? fwd_generic_kernel<T, D, 2> : fwd_generic_kernel<T, D, 1>;
    kernel<<<grid, block, flat_table_bytes(g), stream>>>((const T*)q, (const T*)k, (const T*)v, sel_idx, (T*)out, lse,
                                       g, (uint32_t)(BH / g.kv_group), row_chunks, 32 * nw);
    return hipGetLastError();
}

hipError_t launch_fwd_generic(bool is_bf16, const void* q, const void* k, const void* v,
                              const int32_t* sel_idx, void* out, float* lse, const Geom& g, int D,
                              int64_t BH, hipStream_t stream)
{
#define BSA_CASE(DD)                                                                          \
    case DD:                                                                                  \
        return is_bf16 ? launch_t<uint16_t, DD>(q, k, v, sel_idx, out, lse, g, BH, stream)    \
                       : launch_t<float, DD>(q, k, v, sel_idx, out, lse, g, BH, stream);
    switch (D) {
        BSA_CASE(32)
        BSA_CASE(64)
        BSA_CASE(128)
    }
#undef BSA_CASE
    return hipErrorInvalidValue;
}

}  // namespace bsa
