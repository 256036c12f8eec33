// Host-side launch entry points of the individual kernels; called only by the
// C-ABI layer after it has validated the arguments.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bsa_device.h"

namespace bsa {

// Query blocks ranked per workgroup by the selection kernel; 0 = m too large.
int select_group_size(int m);

hipError_t launch_pool(bool is_bf16, const void* q, const void* k, float* qbar, float* kbar,
                       const Geom& g, int D, int64_t BH, hipStream_t stream);

// Counts, into *n_bad (device), the entries of sel_idx that the attention
// kernels must not be given: out of [0, m), repeated within a row, or (unless
// own_ok) the row's own block.
hipError_t launch_check_selection(const int32_t* sel_idx, int32_t* n_bad, const Geom& g,
                                  bool own_ok, int64_t BH, hipStream_t stream);

// Pooling of Q and K, block scores and top-n as one sequence of launches in
// which the pooling of one part of the batch runs beside the ranking of the part
// before (pooled: qbar, kbar and scratch are there already, only the ranking is
// launched).  The scores of a query block stay in LDS; `scratch` is device memory
// of select_scratch_bytes(...) bytes (BKV = batch * kv_heads): a second copy of
// the pooled keys, per slice [D/4][m][4], which the ranking's threads (one key
// block each) read as consecutive 16-byte groups and launch_pool_select leaves
// there.
size_t select_scratch_bytes(int m, int D, int64_t BKV);
hipError_t launch_pool_select(bool is_bf16, const void* q, const void* k, float* qbar,
                              float* kbar, void* scratch, int32_t* sel_idx, const Geom& g, int D,
                              int64_t BH, bool pooled, hipStream_t stream);

// A launch holds less than 2^32 work items.  Work of `items` of them per slice is
// launched in pieces of whole slices: launch(first slice, slices) returns the status.
template <class F>
inline hipError_t launch_slices(int64_t slices, int64_t items, F launch)
{
    const int64_t fit = (((int64_t)1 << 32) - 1) / items, most = fit < 1 ? 1 : fit;
    for (int64_t first = 0; first < slices; first += most) {
        const hipError_t e = launch(first, slices - first < most ? slices - first : most);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Launches one or two forward jobs of `wgs` workgroups each as one grid (two, where
// one would exceed the 2^32 work items of a launch); launch(job 0, job 1, shape,
// grid) does it.
template <class F>
inline hipError_t launch_jobs(const FwdJob* jobs, int n_jobs, int64_t wgs, int threads, F launch)
{
    const bool together = n_jobs == 2 && 2 * wgs * threads < (int64_t)1 << 32;
    if (wgs >= (int64_t)1 << 31) return hipErrorInvalidValue;
    for (int j = 0; j < n_jobs; j += together ? 2 : 1) {
        const FwdJob &a = jobs[j], &b = together ? jobs[1] : jobs[j];
        launch(a, b,
               FwdShape{{a.n_select, b.n_select}, {a.list_only, b.list_only}, (uint32_t)wgs},
               (unsigned)(together ? 2 * wgs : wgs));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Any tile shape / head dim in {32, 64, 128} / dtype.
hipError_t launch_fwd_generic(bool is_bf16, const void* q, const void* k, const void* v,
                              const FwdJob* jobs, int n_jobs, const Geom& g, int D, int64_t BH,
                              hipStream_t stream);

// bf16 MFMA forward; covers the shapes fwd_mfma_supported() accepts.
bool fwd_mfma_supported(bool is_bf16, const Geom& g, int D);
hipError_t launch_fwd_mfma(const void* q, const void* k, const void* v, const FwdJob* jobs,
                           int n_jobs, const Geom& g, int D, int64_t BH, hipStream_t stream);

// bf16 MFMA forward for head dim 128 (query blocks of 64, 128 or 256 tokens, one
// workgroup of 2, 4 or 8 wavefronts each, K/V tiles shared through LDS).
bool fwd_mfma_d128_supported(bool is_bf16, const Geom& g, int D);
hipError_t launch_fwd_mfma_d128(const void* q, const void* k, const void* v, const FwdJob* jobs,
                                int n_jobs, const Geom& g, int64_t BH, hipStream_t stream);

// What both backward paths need first: delta_l = dO_l . O_l and lse_l * log2(e)
// (fp32, B*heads*N of each; lse null: they are there already), the reverse map of the
// selection in `conn` and, in `order` (int32, key/value slices x m, followed by as many bytes
// of scratch), the order in which the key blocks of each key/value slice are worked on.  It
// is read before dQ is written: dq may serve; null: none is made.  It comes last: `order` may
// lie in the memory of `out`.
hipError_t launch_bwd_prepare(bool is_bf16, const void* out, const void* dout, const float* lse,
                              float* delta, float* lse2, const int32_t* sel_idx, uint32_t* conn,
                              int32_t* order, const Geom& g, int D, int64_t BH, hipStream_t stream);
// A dK/dV launch that runs at once, or nearly, with up to two wavefronts per SIMD needs no
// order of its key blocks: that takes a launch of 4 to 7 us.  How many workgroups run at once
// is the kernel's matter: LDS or registers leave several forms one wavefront per SIMD or half
// of one (the runtime answers in 0.13 us).  With a third more the last ones start where short
// lists have ended, which is soon where all lists are short.  Whole backward, us, ordered | not
// (wavefronts, room):
//   * all at once: 32 blocks of 100 tokens, 4 slices, head dim 32 37.0 | 31.6, 64 46.0 | 41.0; 72
//     of 64, 4 slices 38.5 | 36.6; 128 of 64, 4 slices 73.1 | 61.7; head dim 128, 128 of 128 (1,024)
//     122 | 118; fp32, 128 of 16, 2 slices (512) 95 | 91.
//   * up to a third more, short lists: head dim 32, 128 of 24, 16 slices (2,048, 1,536) 58.4 | 55.2,
//     fp32 128 of 16 92 | 82; head dim 64, 256 of 48, 4 slices 116 | 107, fp32 128 of 16, 7 slices,
//     5 attended (896, 768) 70.7 | 66.2.  Longer ones: fp32 128 of 16, 8 slices, 13 attended (1,024,
//     768) 102 | 105, 128 of 32, 7 attended (2,048, 1,536) 144 | 154; head dim 128, dK/dV of 50
//     of 240, 3 slices, 17 attended (1,200, 1,024) 235 | 255.
//   * half as many more and beyond: head dim 128, 192 of 128 (1,536, 1,024) 155 | 168, 4 heads on 1
//     400 | 458, 192 of 64 117 | 139, 128 of 64, 8 slices (2,048) 226 | 265; fp32 128 of 64, 2 slices
//     323 | 389, 192 of 16, 8 slices (1,536, 512) 300 | 386; head dim 64, fp32 128 of 64 (2,048,
//     1,024) 122 | 137.  Short lists, 4 selected, gain less than it takes: 128 of 48, 6 slices
//     (1,536, 1,024) 110 | 107, of 24 (768, 512) 74 | 71.
//   * more than two wavefronts per SIMD, up to 4,096: 36 of 128, 4 slices 56.7 | 63.4, 288 of 64 in
//     fp32 195 | 229, 72 of 64, 4 slices, 123 | 121.
constexpr int64_t kUnorderedWaves = 2048;
inline bool needs_no_order(int64_t workgroups, int waves, int per_cu, bool short_lists)
{
    const int64_t room = (int64_t)256 * per_cu;
    return workgroups * waves <= kUnorderedWaves &&
           (short_lists ? 3 * workgroups <= 4 * room : workgroups <= room);
}
// In pieces of 32 rows, which take twice as long in fp32 and in proportion to the head dim.
inline bool short_lists(const Geom& g, int D, bool is_f32)
{
    const int64_t rows = (int64_t)g.kv_group * (g.n_select + 1 - g.list_only) * g.block_tokens;
    return rows * D * (is_f32 ? 2 : 1) <= 24 * 32 * 32;
}
// Lists of one length need none at all: the local branch's, and without selected blocks (fp32, 180
// blocks of 30, 4 slices, head dim 128 59.9 | 54.7).
inline bool even_lists(const Geom& g) { return g.add_dk || g.n_select == 0; }
template <class K>
inline bool needs_no_order(K kernel, int64_t workgroups, int waves, size_t dynamic_lds,
                           bool short_lists)
{
    int per_cu = 0;
    if (!needs_no_order(workgroups, waves, 8, short_lists)) return false;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kernel, 64 * waves,
                                                     dynamic_lds) != hipSuccess) {
        (void)hipGetLastError();                      // (not the launch's)
        return false;
    }
    return needs_no_order(workgroups, waves, per_cu, short_lists);
}

// Backward with the selection fixed, any tile shape / head dim in {32, 64, 128} /
// dtype.  `delta` and `lse2` are fp32 scratch of B*heads*N floats each, `conn`
// scratch of bwd_connection_words(...) 32-bit words (the reverse map of the
// selection: one bit per (query slice, key block, query block)).  lse == nullptr: delta
// and lse2 are there already.  order == nullptr: dQ is computed before dK and dV, which
// may then be written over k and v (a workgroup reads only the rows that it writes).
inline int64_t bwd_connection_words(int m, int64_t BH) { return BH * m * (int64_t)((m + 31) >> 5); }
hipError_t launch_bwd(bool is_bf16, const void* q, const void* k, const void* v, const void* out,
                      const float* lse, const void* dout, const int32_t* sel_idx, void* dq,
                      void* dk, void* dv, float* delta, float* lse2, uint32_t* conn, int32_t* order,
                      const Geom& g, int D, int64_t BH, hipStream_t stream);

// bf16 MFMA backward (head dim 64 or 128, blocks of 64, 128 or 256 tokens), same
// scratch.
bool bwd_mfma_supported(bool is_bf16, const Geom& g, int D);
hipError_t launch_bwd_mfma(const void* q, const void* k, const void* v, const void* out,
                           const float* lse, const void* dout, const int32_t* sel_idx, void* dq,
                           void* dk, void* dv, float* delta, float* lse2, uint32_t* conn, int32_t* order,
                           const Geom& g, int D, int64_t BH, hipStream_t stream);

// The block-level part of the three-branch output: pooled q, k, v, the selection
// (as launch_pool_select), the coarse branch (softmax over all pooled key blocks
// times pooled values, fp32 [B*heads, m, D]) and the block lists of the local branch
// (int32 [B*heads, m, local_h*local_w - 1]).  kbar_il: the channel-interleaved copy
// of the pooled keys (the scratch of launch_pool_select).
hipError_t launch_blocks_three_branch(bool is_bf16, const void* q, const void* k, const void* v,
                                      float* qbar, float* kbar, float* vbar, float* kbar_il,
                                      int32_t* sel_idx, float* obar, int32_t* lists, int local_h,
                                      int local_w, const Geom& g, int D, int64_t BH,
                                      hipStream_t stream);
hipError_t launch_coarse(const float* qbar, const float* kbar_il, const float* vbar, float* obar,
                         const Geom& g, int D, int64_t BH, hipStream_t stream);

// The gated sum of the three branches.
hipError_t launch_combine(bool is_bf16, const float* obar, const void* o_fg, const void* o_l,
                          const float* gates, void* out, const Geom& g, int D, int64_t BH,
                          hipStream_t stream);

// Backward of the three-branch output: upstream gradients, delta and lse2 of the two
// attention branches, the gate gradients and the gated block sums of dout; the coarse
// branch's gradients on the pooled tensors, chunk_rows query blocks at a time (a_mat,
// ds_mat: fp32 scratch [B*heads, chunk_rows, m]; kbar_il: see launch_pool_select).
int coarse_bwd_group_size(int m, int D);
struct BranchGrads {
    const float* obar;                          // coarse rows
    const void *o_fg, *o_l;                     // branch outputs
    const float *lse_fg, *lse_l, *gates;
    const void* dout;
    void *do_fg, *do_l;                         // out: upstream gradients of the branches
    float *dgates, *dobar;                      // out
    float *delta_fg, *delta_l, *lse2_fg, *lse2_l;    // out: see launch_bwd_prepare
};
hipError_t launch_branch_grads(bool is_bf16, const BranchGrads& x, const Geom& g, int D, int64_t BH,
                               hipStream_t stream);
hipError_t launch_coarse_bwd(const float* qbar, const float* kbar, const float* kbar_il,
                             const float* vbar, const float* dobar, float* a_mat, float* ds_mat, float* dqbar,
                             float* dkbar, float* dvbar, const Geom& g, int D, int64_t BH,
                             int chunk_rows, hipStream_t stream);

// Measurement aid: `workgroups` x 4 wavefronts, each issuing 16 * iters
// v_mfma_f32_32x32x16_bf16 on register operands; sink: workgroups * 256 floats.
hipError_t launch_mfma_probe(float* sink, int workgroups, int iters, hipStream_t stream);

}  // namespace bsa
