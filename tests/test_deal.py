"""Which workgroup works on what (csrc/bsa_deal.h), compiled for the host: every item once,
and what shares an L2 lies on one XCD.  Workgroup w runs on XCD w % 8."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_16429_amd", "csrc")

SOURCE = """
#include "bsa_launch.h"
using namespace bsa;
extern "C" void deal_of(int64_t slice_bytes, int block_tokens, int32_t* out)
{
    const Deal d = xcd_deal(slice_bytes, block_tokens);
    out[0] = d.whole_slices;
    out[1] = d.run_log2;
}
extern "C" void key_deal_of(int64_t slice_bytes, int block_tokens, int ordered, int even,
                            int32_t* out)
{
    const Deal d = key_deal(xcd_deal(slice_bytes, block_tokens), slice_bytes, ordered, even);
    out[0] = d.whole_slices;
    out[1] = d.run_log2;
}
extern "C" int no_order(int64_t workgroups, int waves, int per_cu, int short_lists)
{
    return needs_no_order(workgroups, waves, per_cu, short_lists);
}
extern "C" void map_all(int whole, int run_log2, uint32_t blocks, uint32_t heads,
                        uint32_t chunks, uint32_t n_units, uint32_t* out)
{
    const uint32_t all = n_units * heads * blocks * chunks;
    for (uint32_t w = 0; w < all; ++w)
        map_unit(Deal{whole, run_log2}, w, blocks, heads, chunks, n_units,
                 out[3 * w], out[3 * w + 1], out[3 * w + 2]);
}
"""


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    d = tmp_path_factory.mktemp("deal")
    src, lib = d / "deal.hip", d / "deal.so"
    src.write_text(SOURCE)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950",
                    "--offload-host-only", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", str(lib)], check=True)
    lib = ctypes.CDLL(str(lib))
    lib.no_order.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 3
    lib.deal_of.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_void_p]
    lib.key_deal_of.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 3 + [ctypes.c_void_p]
    return lib


def mapped(deal, whole, run_log2, blocks, heads, chunks, n_units):
    """[workgroups, 3]: key/value slice, query head of the slice, item of the head."""
    out = np.empty((n_units * heads * blocks * chunks, 3), dtype=np.uint32)
    deal.map_all(whole, run_log2, blocks, heads, chunks, n_units, out.ctypes.data_as(ctypes.c_void_p))
    return out.astype(np.int64)


@pytest.mark.parametrize("seed", range(4))
def test_every_item_once(deal, seed):
    rng = random.Random(seed)
    for _ in range(300):
        whole, run_log2 = rng.randint(0, 1), rng.randint(0, 7)
        blocks, n_units = rng.randint(1, 200), rng.randint(1, 20)
        heads, chunks = rng.choice([1, 1, 2, 3, 4, 7]), rng.choice([1, 1, 2, 3, 4, 5, 8])
        m = mapped(deal, whole, run_log2, blocks, heads, chunks, n_units)
        per_head = blocks * chunks
        assert m[:, 1].max() < heads and m[:, 2].max() < per_head
        key = np.sort((m[:, 0] * heads + m[:, 1]) * per_head + m[:, 2])
        assert np.array_equal(key, np.arange(len(m)))


@pytest.mark.parametrize("heads,blocks,chunks,n_units,run_log2", [
    (4, 128, 1, 1, 8),      # an eighth to each XCD
    (8, 450, 1, 2, 8),
    (4, 24, 2, 5, 7),
    (3, 2025, 1, 1, 7),     # runs of 128 and a tail
    (4, 4050, 3, 3, 6),
])
def test_heads_of_a_slice_share_an_xcd(deal, heads, blocks, chunks, n_units, run_log2):
    """Of the slices that all XCDs share, an XCD works on the same items of all query heads of a
    slice, but for the ends of its runs."""
    m = mapped(deal, 0, run_log2, blocks, heads, chunks, n_units)
    xcds = {}
    for w, (unit, _, item) in enumerate(m):
        xcds.setdefault((unit, item), set()).add(w % 8)
    spread = sum(len(x) > 1 for x in xcds.values())
    runs = heads * blocks * n_units // (1 << run_log2) + 8
    assert spread <= chunks * runs, f"{spread} of {len(xcds)} items on more than one XCD"


@pytest.mark.parametrize("blocks,heads,chunks,n_units,run_log2", [
    (128, 1, 4, 1, 0),     # key blocks, one by one
    (225, 1, 2, 3, 0),
    (96, 1, 3, 7, 0),
    (1024, 1, 2, 1, 6),    # runs of 64
    (700, 2, 5, 3, 5),
])
def test_chunks_of_a_block_share_an_xcd(deal, blocks, heads, chunks, n_units, run_log2):
    """The workgroups of one block, which gather the same tiles, follow each other on one XCD, but
    for the blocks that the eighths of the last round cut (seven)."""
    m = mapped(deal, 0, run_log2, blocks, heads, chunks, n_units)
    xcds = {}
    for w, (unit, head, item) in enumerate(m):
        xcds.setdefault((unit, head, item // chunks), []).append(w)
    apart = sum(not np.array_equal(x, x[0] + 8 * np.arange(chunks)) for x in xcds.values())
    assert apart <= 7, f"{apart} of {len(xcds)} blocks on more than one XCD"


@pytest.mark.parametrize("megabytes,whole", [(1, 1), (32, 1), (33, 0), (265, 0)])
def test_deal_of_query_blocks(deal, megabytes, whole):
    """Slices up to 32 MB whole, larger ones in runs of about 16,384 tokens."""
    d = np.empty(2, dtype=np.int32)
    for block_tokens, run in ((1, 16384), (60, 256), (64, 256), (100, 128), (256, 64), (1024, 16)):
        deal.deal_of(megabytes << 20, block_tokens, d.ctypes.data)
        assert d.tolist() == [whole, run.bit_length() - 1]


@pytest.mark.parametrize("megabytes", [1, 31, 33, 64, 265, 2048])
@pytest.mark.parametrize("block_tokens", [64, 100, 256])
def test_deal_of_key_blocks(deal, megabytes, block_tokens):
    """Slices whose key blocks are ordered, or have lists of one length, go to one XCD whatever
    their size; only lists of one length go in runs, those of the query blocks."""
    d = np.empty((4, 2), dtype=np.int32)
    deal.deal_of(megabytes << 20, block_tokens, d[0].ctypes.data)
    for row, (ordered, even) in zip(d[1:], ((1, 0), (0, 1), (0, 0))):
        deal.key_deal_of(megabytes << 20, block_tokens, ordered, even, row.ctypes.data)
    assert d[1].tolist() == [1, 0]
    assert d[2].tolist() == [1, d[0, 1]]
    assert d[3].tolist() == [int(megabytes <= 32), 0]


@pytest.mark.parametrize("waves,per_cu", [
    (1, 2), (2, 1), (4, 1), (2, 3), (4, 2), (8, 1), (3, 1), (2, 8)])
def test_launches_without_an_order(deal, waves, per_cu):
    """dK/dV goes without an order only where 256 CUs that hold per_cu workgroups each take the launch
    at once, or all but a quarter of it where lists are short, and at two wavefronts per SIMD at
    most."""
    for short, room in ((0, 256 * per_cu), (1, 256 * per_cu * 4 // 3)):
        most = min(room, 2048 // waves)
        assert deal.no_order(most, waves, per_cu, short)
        assert not deal.no_order(most + 1, waves, per_cu, short)


def test_whole_slices(deal):
    """Eight slices at a time, one to each XCD."""
    m = mapped(deal, 1, 6, 25, 3, 2, 19)
    dealt = m[: 16 * 150]
    assert np.array_equal(dealt[:, 0] % 8, np.arange(len(dealt)) % 8)
    assert m[16 * 150 :, 0].min() == 16
