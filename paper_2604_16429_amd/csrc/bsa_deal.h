// Which workgroup works on what (host and device; tested on the CPU).  Workgroup ids go
// round-robin over the 8 XCDs, each with its own L2; what the workgroups of an XCD that run
// at the same time gather in common is fetched into that L2 once.
//   * Slices whose K and V take up to 32 MB: dealt to XCDs whole, key/value slice u to
//     XCD u % 8, the items of the query heads that share it back to back.  Eight of them
//     fit the 256 MB of cache behind the L2s.
//   * Larger ones, and the last (number of key/value slices % 8): all XCDs share a slice,
//     in runs of consecutive blocks dealt to them in turn.  Near query blocks attend to the
//     same blocks, so that a run finds them in its L2, and the runs that are worked on
//     at the same time keep to one region of one slice, which the cache behind holds.  A run
//     takes the same blocks of all query heads that share the slice: head after head, the
//     part of the slice that an XCD needs was fetched by as many XCDs as there are heads, and
//     small launches were slower than item by item.
//   * The workgroups of one block (its row chunks) stay together: they gather the same tiles.
//     Key blocks, whose chunks walk the same list, dealt workgroup by workgroup | block by
//     block, backward us: 1 slice of 128 blocks of 256 in four chunks 129 | 122, 2 slices 183 | 178,
//     3 with 6 heads 454 | 444, head dim 128 347 | 338; 1,024 tokens, 3 with 6 heads 5,190 | 4,961.
// Forward us, dealt item by item before (small numbers of slices) | in runs: 6 slices of 2,276
// blocks of 64, 31 attended, head dim 128, 24 heads 7,040 | 3,960; 4 of 450 blocks of 64 57 |
// 45; 15 of 450 106 | 97; 2 of 1,800, 6 heads 321 | 280; 3 of 384 of 128, 12 heads 517 | 493; 4 of
// 4,050 of 256 4,670 | 4,710.  One run per XCD: the last 4,920 (the eight regions do not
// fit the cache, and the slowest one is waited for).
// Heads that share a slice, item by item | in runs head after head | in runs of all heads, head
// dim 64, blocks of 64, slices x blocks, query heads: 1 x 128, 8 17.6 | 19.3 | 17.7; 2 x 128, 8
// 18.2 | 19.3 | 17.6; 3 x 288, 12 52.7 | 53.6 | 50.3; 3 x 450, 12 87.4 | 81.8 | 76.4; 7 x 450, 14
// 107 | 97 | 92; head dim 128: 4 x 4,050, 16 2,565 | 1,902 | 1,765.
// 16 slices, dealt whole | in runs: 4,050 of 256 (265 MB) 20,440 | 19,190, at head dim 128
// 22,980 | 22,330; 2,025 of 128 (66 MB) 1,528 | 1,458; 3,422 (112 MB) 2,429 | 2,376; 1,800 of
// 64 at head dim 128 (59 MB) 1,853 | 1,872; 32 slices of 450 of 64 (7 MB) 1,257 | 1,287; 72 of
// 384 of 128 (13 MB) 11,700 | 11,930.  Just above 32 MB it is 2 % either way: 8 of 1,056 of
// 128 (35 MB) 364 | 368; 16 of 1,152 (38 MB) 797 | 797, 32 heads on 8 1,586 | 1,549; 16 of 600
// of 256 (39 MB) 1,467 | 1,458; at head dim 128 16 of 1,200 of 64 (39 MB) 583 | 594, of 600 of
// 128 835 | 823.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bsa {

struct Deal {
    int32_t whole_slices;      // slices are dealt to XCDs whole while there are eight
    int32_t run_log2;          // blocks of a run (of any head)
};

// Workgroup w of a launch over n_units key/value slices -> slice, query head (of the `heads`
// that share it) and item of that head: `chunks` items to each of `blocks` blocks.
__host__ __device__ __forceinline__ void map_unit(Deal deal, uint32_t w, uint32_t blocks,
                                                  uint32_t heads, uint32_t chunks,
                                                  uint32_t n_units, uint32_t& unit,
                                                  uint32_t& head, uint32_t& item)
{
    const uint32_t per_head = blocks * chunks, per_unit = per_head * heads;
    const uint32_t units_dealt = deal.whole_slices ? n_units & ~7u : 0;
    const uint32_t dealt = units_dealt * per_unit;
    if (w < dealt) {
        const uint32_t seq = w >> 3, round = seq / per_unit, r = seq - round * per_unit;
        unit = round * 8 + (w & 7);
        head = heads == 1 ? 0 : r / per_head;
        item = r - head * per_head;
        return;
    }
    // runs for all XCDs while there are, then an eighth of what is left to each
    const int log2 = deal.run_log2;
    const uint32_t rest = (n_units - units_dealt) * blocks * heads;
    const uint32_t even = (rest >> (log2 + 3) << (log2 + 3)) * chunks, tail = rest * chunks - even;
    const uint32_t xcd = (w - dealt) & 7, seq = (w - dealt) >> 3;
    uint32_t at;
    if (w - dealt < even) {
        const uint32_t place = seq / chunks;
        at = ((((place >> log2 << 3) + xcd) << log2) + (place & ((1u << log2) - 1))) * chunks +
             (seq - place * chunks);
    } else {
        at = even + (seq - (even >> 3)) + xcd * (tail >> 3) + (xcd < (tail & 7u) ? xcd : tail & 7u);
    }
    const uint32_t u = at / per_unit, r = at - u * per_unit;
    unit = units_dealt + u;
    head = 0;
    item = r;
    if (heads > 1) {                                 // the heads of a block side by side
        const uint32_t of_block = heads * chunks, block = r / of_block;
        const uint32_t in_block = r - block * of_block;
        head = in_block / chunks;
        item = block * chunks + (in_block - head * chunks);
    }
}

// Runs of about 16,384 tokens (of one head or another), from 16 blocks of 1,024 tokens to 16,384
// of one: 2 slices of 1,800 blocks of 64 in runs of
// 4,096 300 us, of 8,192 283, of 16,384 280, of 65,536 283.
inline Deal xcd_deal(int64_t slice_bytes, int block_tokens)
{
    Deal d;
    d.whole_slices = slice_bytes <= (int64_t)32 << 20;
    d.run_log2 = 14;
    for (int rows = block_tokens - 1; rows > 0; rows >>= 1) --d.run_log2;
    return d;
}

// Key blocks (dK and dV).  `ordered`: in the order of their lists, long ones first; `even`: all
// lists are as long (local branch); neither: uneven lists as they lie.
//   * Ordered or even, slices are dealt to XCDs whole whatever their size: an XCD then gathers
//     the query tiles of its own slice, and the long lists of all slices start early.  Shared
//     block by block, each tile was fetched into eight L2s and the long lists of the last slice
//     came last.  Whole backward, us, slices above 32 MB shared | whole: fp32, 8 slices of
//     1,200 blocks of 64 (38 MB) 2,928 | 2,665, of 1,024 of 128 (64 MB) 9,063 | 8,446; bf16, 8 of
//     1,600 of 10 x 10 (39 MB) 2,278 | 2,116, of 1,200 of 64 at head dim 128 (38 MB) 1,479 | 1,356;
//     local branch, 8 of 4,096 of 128 (128 MB) 15,500 | 15,020.  Many blocks in bf16 lose a little: 8
//     of 2,048 of 128 2,497 | 2,504, 16 of 4,050 of 256 38,250 | 38,470, 16 selected 67,800 | 68,420,
//     20 of 8,100 of 64 3,819 | 3,898.
//   * Uneven lists as they lie balance best block by block over all XCDs: above 32 MB, gradients
//     in place, head dim 128, 8 slices of 42 MB 1,572, whole 1,650, 64 MB 2,679 | 2,663, fp32
//     9,087 | 9,150.  Below, 0.92 to 1.07 times either way.
//   * What is left is shared block by block: runs would give one XCD all the long lists (1 slice
//     of 225 blocks of 128 in runs 84 us, block by block 70).  Even lists: in runs as the query
//     blocks are (6 slices of 450 blocks, backward of three branches 394 | 389).
inline Deal key_deal(Deal d, int64_t slice_bytes, bool ordered, bool even)
{
    d.whole_slices = ordered || even || slice_bytes <= (int64_t)32 << 20;
    if (!even) d.run_log2 = 0;
    return d;
}

}  // namespace bsa
