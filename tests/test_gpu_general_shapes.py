"""GPU parity of the general-shape kernels at the sizes where their tiling can go
wrong: block sizes around the 32-row wavefront tile and the 256-row workgroup,
key sequences around the 32- and 64-key tiles (block boundaries inside a tile,
a last tile of one key), lists around the 64 blocks that are sorted and the
1,024 that the LDS table holds."""
import numpy as np
import pytest
import torch

from inputs.fields import round_to_bf16
from tests.helpers import rand_qkv, random_selection, shape_ns

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util
    return gpu_util


SHAPES = [
    # H, W, bh, bw, D, n
    (8, 12, 1, 1, 32, 7),        # b = 1: every key its own block
    (9, 12, 3, 3, 64, 6),        # b = 9: 63 keys, a tile minus one
    (10, 13, 5, 1, 128, 12),     # b = 5: 65 keys, a last tile of one key
    (10, 9, 2, 3, 64, 15),       # n = m: everything, b = 6, grid no multiple of 8
    (31, 8, 31, 1, 64, 2),       # b = 31: one wavefront with an idle row
    (22, 33, 11, 3, 32, 3),      # b = 33: two wavefronts, one row in the second
    (16, 30, 8, 15, 128, 3),     # b = 120
    (14, 57, 7, 19, 64, 4),      # b = 133: five wavefronts
    (32, 40, 16, 20, 32, 1),     # b = 320: two workgroups of five wavefronts per block
    (34, 60, 17, 30, 64, 2),     # b = 510: two workgroups of eight, two idle rows
    (20, 26, 2, 2, 64, 63),      # 64 attended blocks: the last list that is sorted
    (20, 26, 2, 2, 64, 64),      # 65: kept in the given order
    (16, 30, 16, 1, 64, 5),      # b = 16: one fp32 wavefront of 16 rows
    (34, 12, 17, 1, 128, 4),     # b = 17: one row in the second of them
    (24, 36, 8, 6, 64, 7),       # b = 48: three, two of which gather; bf16 two, the second
                                 # 16 rows wide
    (20, 50, 10, 10, 32, 5),     # b = 100: the fourth of four 16 rows wide
    (28, 30, 7, 10, 128, 5),     # b = 70: the third of three
    (46, 48, 1, 2, 32, 959),     # list and its repeated last entry just fit the LDS table
    (46, 48, 1, 2, 32, 960),     # just not
    (46, 48, 1, 2, 32, 1030),    # more listed blocks than the LDS table holds
]


def inputs_of(cfg, seed):
    q, k, v = rand_qkv(cfg, seed)
    if cfg.dtype == "bf16":
        q, k, v = (round_to_bf16(x) for x in (q, k, v))
    return q, k, v


def times(cfg, groups, *tensors):
    """One entry as often as it takes for a launch of up to 256 row wavefronts, of up to 512
    or more, which is where four, two groups or one take the keys of long enough lists."""
    rows, most = (16, 4 if cfg.head_dim == 32 else 8) if cfg.dtype == "fp32" else (32, 8)
    tiles = -(-cfg.block_tokens // rows)
    chunks = -(-tiles // most)
    per_entry = cfg.heads * cfg.n_blocks * chunks * -(-tiles // chunks)
    cfg.batch = {4: 256 // per_entry, 2: 512 // per_entry, 1: 512 // per_entry + 1}[groups]
    low, high = {4: (0, 256), 2: (256, 512), 1: (512, 1 << 30)}[groups]
    assert low < cfg.batch * per_entry <= high
    return [np.repeat(x, cfg.batch, axis=0) for x in tensors]


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("H,W,bh,bw,D,n", SHAPES)
def test_general_forward(G, oracle, large, dtype, H, W, bh, bw, D, n):
    """large: the entry as often as it takes for the workgroups of a launch that does not
    split the keys.  fp32: 1e-5 of the largest output, lse likewise.  bf16: the output is one
    rounding (half an ulp: at most 2^-8 of the value) of a sum whose weights are
    kept as two bf16 terms (truncated to 2^-7, the rest rounded to 2^-8 of itself:
    2^-15 of the largest value; twice that covers the fp32 sums as well)."""
    cfg = shape_ns(1, 2, H, W, bh, bw, D, min(n, (H // bh) * (W // bw) - 1), dtype)
    q, k, v = inputs_of(cfg, 40 + H + W + D)
    s = oracle.shape_of(cfg)
    idx = random_selection(cfg, 7)
    out_ref, lse_ref = oracle.fwd(s, q, k, v, idx)
    out, lse = G.gpu_fwd(cfg, *(times(cfg, 1, q, k, v, idx) if large else (q, k, v, idx)))
    err = np.abs(out - out_ref)
    if dtype == "fp32":
        assert err.max() <= 1e-5 * np.abs(out_ref).max()
    else:
        assert (err <= 2.0 ** -8 * np.abs(out_ref) + 2.0 ** -14 * np.abs(v).max()).all()
    assert np.abs(lse - lse_ref).max() <= 1e-5 * max(1.0, np.abs(lse_ref).max())


@pytest.mark.parametrize("groups", [4, 2, 1])
@pytest.mark.parametrize("dtype,H,W,bh,bw,D,n", [
    ("fp32", 9, 12, 3, 3, 64, 6),          # 63 keys: two tiles, in two groups
    ("fp32", 10, 20, 5, 5, 32, 7),         # 200: seven, the last round of four not full
    ("bf16", 16, 28, 8, 7, 32, 7),         # 448: seven
    ("bf16", 12, 30, 2, 15, 64, 7),        # 240: four, in two groups of one wavefront
    ("fp32", 22, 33, 11, 3, 32, 13),       # b = 33
    ("bf16", 22, 33, 11, 3, 64, 13),
    ("fp32", 14, 57, 7, 19, 64, 4),        # b = 133
    ("bf16", 16, 60, 8, 15, 64, 4),        # b = 120
    ("fp32", 16, 28, 8, 7, 128, 7),        # two groups at the most
    ("bf16", 16, 28, 8, 7, 128, 7),
    ("fp32", 12, 44, 2, 4, 32, 64),        # 65 listed blocks: in the given order
    ("bf16", 12, 44, 2, 4, 32, 64),
])
def test_general_forward_key_split(G, oracle, dtype, groups, H, W, bh, bw, D, n):
    """Launches that take the keys in four groups, two or one.  All copies of the entry
    agree exactly, and with the oracle as in test_general_forward; the bits tell that the
    small launches did split (see test_general_forward_unsplit_small_launches) and stay
    within those bounds of the large launch's (bf16: two roundings of the output)."""
    cfg = shape_ns(1, 1, H, W, bh, bw, D, min(n, (H // bh) * (W // bw) - 1), dtype)
    q, k, v = inputs_of(cfg, 70 + H + W + D)
    idx = random_selection(cfg, 9)
    out_ref, lse_ref = oracle.fwd(oracle.shape_of(cfg), q, k, v, idx)
    out, lse = G.gpu_fwd(cfg, *times(cfg, groups, q, k, v, idx))
    assert cfg.batch > 1 and (out == out[:1]).all() and (lse == lse[:1]).all()
    err, top = np.abs(out[:1] - out_ref), np.abs(out_ref).max()
    if dtype == "fp32":
        assert err.max() <= 1e-5 * top
    else:
        assert (err <= 2.0 ** -8 * np.abs(out_ref) + 2.0 ** -14 * np.abs(v).max()).all()
    assert np.abs(lse[:1] - lse_ref).max() <= 1e-5 * max(1.0, np.abs(lse_ref).max())
    whole = G.gpu_fwd(cfg, *times(cfg, 1, q, k, v, idx))
    assert np.array_equal(whole[1][0], lse[0]) == (groups == 1)
    apart = np.abs(whole[0][0] - out[0])
    if dtype == "fp32":
        assert apart.max() <= 1e-5 * top
    else:
        assert (apart <= 2.0 ** -7 * np.abs(out_ref) + 2.0 ** -13 * np.abs(v).max()).all()


@pytest.mark.parametrize("groups", [4, 2, 1])
@pytest.mark.parametrize("dtype,D", [("fp32", 32), ("fp32", 64), ("fp32", 128),
                                     ("bf16", 32), ("bf16", 64), ("bf16", 128)])
def test_general_forward_rising_maxima(G, oracle, dtype, D, groups):
    """Scores of up to about 80 whose maxima grow with the block index, so that the
    reference of the softmax moves at most tiles.  A score is off by up to
    2^-24 (sqrt(D / 12) + 1) of its value, 2.1e-5, and a weight by that of two: 1e-4 of the
    largest output (bf16: on top of the bound of test_general_forward) and of lse."""
    cfg = shape_ns(1, 1, 24, 36, 6, 6, D, 15, dtype)
    q, k, v = inputs_of(cfg, 33 + D)
    grow = (1.0 + 6.0 * np.arange(24) / 23).astype(np.float32).reshape(4, 1, 6, 1, 1)
    k = (k.reshape(4, 6, 6, 6, D) * grow).reshape(k.shape)
    q = 3.0 * q
    if dtype == "bf16":
        q, k = round_to_bf16(q), round_to_bf16(k)
    idx = random_selection(cfg, 34)
    out_ref, lse_ref = oracle.fwd(oracle.shape_of(cfg), q, k, v, idx)
    assert np.abs(lse_ref).max() > 40.0
    out, lse = G.gpu_fwd(cfg, *times(cfg, groups, q, k, v, idx))
    err, bound = np.abs(out - out_ref), 1e-4 * np.abs(out_ref).max()
    if dtype == "bf16":
        bound = bound + 2.0 ** -8 * np.abs(out_ref) + 2.0 ** -14 * np.abs(v).max()
    assert (err <= bound).all()
    assert np.abs(lse - lse_ref).max() <= 1e-4 * max(1.0, np.abs(lse_ref).max())


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("mask", [-1e10, -1e30, -3e38])
@pytest.mark.parametrize("dtype,H,W,bh,bw,D", [
    ("fp32", 10, 20, 5, 5, 32), ("fp32", 16, 32, 8, 8, 64), ("fp32", 10, 20, 5, 5, 128),
    ("bf16", 16, 32, 8, 8, 32), ("bf16", 10, 20, 5, 5, 64), ("bf16", 10, 20, 5, 5, 128),
])
def test_general_forward_finite_masks(G, oracle, dtype, H, W, bh, bw, D, mask, large):
    """Keys masked by a large finite score through a channel of their own.  Masked: the
    first tiles of a row, the last ones, and all of them (block 0: the weights are
    then equal; only for masks beside which the other channels vanish in 64 bits as
    they do in 32).  `large` and bounds as in test_general_forward."""
    cfg = shape_ns(1, 2, H, W, bh, bw, D, 2, dtype)
    q, k, v = inputs_of(cfg, 3 + D)
    rows, cols = H // bh, W // bw
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    grid = k.reshape(1, 2, rows, bh, cols, bw, D)            # blocks 0, 1, 2 are masked
    grid[:, :, 0, :, :3, :, 0] = mask
    if dtype == "bf16":
        k = round_to_bf16(k)
    idx = random_selection(cfg, 5)
    idx[:, :, 0] = [1, 2]
    idx[:, :, 1] = [0, cols]
    idx[:, :, cols] = [0, cols + 1]
    out_ref, lse_ref = oracle.fwd(oracle.shape_of(cfg), q, k, v, idx)
    out, lse = G.gpu_fwd(cfg, *(times(cfg, 1, q, k, v, idx) if large else (q, k, v, idx)))
    keep = np.ones((H, W), dtype=bool)
    if mask > -1e20:
        keep[:bh, :bw] = False
    keep = keep.reshape(-1)
    err, ref = np.abs(out - out_ref)[:, :, keep], np.abs(out_ref)[:, :, keep]
    if dtype == "fp32":
        assert err.max() <= 1e-5 * ref.max()
    else:
        assert (err <= 2.0 ** -8 * ref + 2.0 ** -14 * np.abs(v).max()).all()
    lse_err = np.abs(lse - lse_ref) / np.maximum(1.0, np.abs(lse_ref))
    assert lse_err[:, :, keep].max() <= 1e-5
    assert np.isfinite(out).all() and np.isfinite(lse).all()


@pytest.mark.parametrize("groups", [4, 2, 1])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_general_forward_nan_keys(G, dtype, groups):
    """A row that attends to a block of NaN keys (values finite) becomes NaN, whatever the
    place of the block in the row's list and the size of the launch; the others do not."""
    cfg = shape_ns(1, 1, 32, 32, 8, 8, 32, 8, dtype)
    q, k, v = inputs_of(cfg, 11)
    k[0, 0].reshape(4, 8, 4, 8, 32)[1, :, 2] = np.nan        # block 6
    idx = random_selection(cfg, 12)
    out, lse = G.gpu_fwd(cfg, *times(cfg, groups, q, k, v, idx))
    sees = (idx[0, 0] == 6).any(axis=1) | (np.arange(16) == 6)
    sees = np.broadcast_to(sees.reshape(4, 1, 4, 1), (4, 8, 4, 8)).reshape(-1)
    assert (np.isnan(lse) == sees).all() and (np.isnan(out) == sees[:, None]).all()


@pytest.mark.parametrize("groups", [4, 2, 1])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_general_forward_masks_past_the_range(G, oracle, dtype, groups):
    """Keys masked by a score of -3e38, which times log2(e) leaves the range of fp32, as the
    first keys of a row, the first that a group takes and others: weight 0.  Bounds of
    test_general_forward."""
    cfg = shape_ns(1, 1, 32, 32, 8, 8, 32, 8, dtype)
    q, k, v = (0.4 * x for x in inputs_of(cfg, 13))
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    keys = k[0, 0].reshape(4, 8, 4, 8, 32)
    keys[0, :, :, :, 0] = -3e38                              # blocks 0 to 3
    keys[2, :4, 1, :, 0] = -3e38                             # half of block 9
    if dtype == "bf16":
        q, k, v = (round_to_bf16(x) for x in (q, k, v))
    idx = random_selection(cfg, 14)
    out_ref, lse_ref = oracle.fwd(oracle.shape_of(cfg), q, k, v, idx, 1.0)
    out, lse = G.gpu_fwd(cfg, *times(cfg, groups, q, k, v, idx), softmax_scale=1.0)
    err = np.abs(out - out_ref)
    if dtype == "fp32":
        assert err.max() <= 1e-5 * np.abs(out_ref).max()
    else:
        assert (err <= 2.0 ** -8 * np.abs(out_ref) + 2.0 ** -14 * np.abs(v).max()).all()
    assert np.abs(lse - lse_ref).max() <= 1e-5 * max(1.0, np.abs(lse_ref).max())


@pytest.mark.parametrize("dtype,groups,H,W,bh,bw,D,n", [
    ("fp32", 2, 16, 32, 4, 4, 128, 20),      # one row wavefront per block: no pairs, and
    ("bf16", 2, 16, 32, 4, 4, 128, 20),      # more workgroups than CUs
    ("fp32", 2, 12, 48, 6, 6, 128, 9),       # three
    ("fp32", 2, 12, 48, 6, 6, 64, 9),
    ("fp32", 2, 16, 32, 4, 4, 32, 13),       # 7 tiles at head dim 32
    ("bf16", 4, 16, 32, 8, 8, 32, 2),        # 3 tiles
    ("bf16", 2, 16, 32, 8, 8, 32, 2),
    ("bf16", 4, 12, 24, 6, 6, 64, 4),
    ("bf16", 2, 12, 24, 6, 6, 128, 4),
])
def test_general_forward_unsplit_small_launches(G, dtype, groups, H, W, bh, bw, D, n):
    """Launches that do not split the keys although they are small: the bits of a large
    one."""
    cfg = shape_ns(1, 1, H, W, bh, bw, D, n, dtype)
    inputs = *inputs_of(cfg, 21), random_selection(cfg, 22)
    large = G.gpu_fwd(cfg, *times(cfg, 1, *inputs))
    small = G.gpu_fwd(cfg, *times(cfg, groups, *inputs))
    assert all(np.array_equal(x[0], y[0]) for x, y in zip(small, large))


@pytest.mark.parametrize("dtype,kv_heads", [("fp32", 0), ("bf16", 0), ("fp32", 1), ("bf16", 1)])
@pytest.mark.parametrize("H,W,bh,bw,D,n", SHAPES)
def test_general_backward(G, oracle, dtype, kv_heads, H, W, bh, bw, D, n):
    """fp32: 1e-4 of the largest entry, the bound of the other fp32 backward tests.
    bf16: the stored gradient is off by half an ulp (2^-8 of its value, 4e-3) and
    delta = dO . O by the rounding of O (2^-8 of O, D zero-mean terms: about 2^-8
    sqrt(D) |dO| |O| <= 0.01 here, which enters dS weighted with P <= 1 and the
    softmax scale): 1e-2 of max(1, largest entry) covers both.  Reruns are bitwise
    identical."""
    cfg = shape_ns(1, 2, H, W, bh, bw, D, min(n, (H // bh) * (W // bw) - 1), dtype, kv_heads)
    rng = np.random.default_rng(90 + H + W + D)
    shape = (1, 2, H * W, D)
    q, dout = (rng.standard_normal(shape).astype(np.float32) for _ in range(2))
    k, v = (rng.standard_normal((1, kv_heads or 2, H * W, D)).astype(np.float32) for _ in range(2))
    if dtype == "bf16":
        q, k, v, dout = (round_to_bf16(x) for x in (q, k, v, dout))
    s = oracle.shape_of(cfg)
    idx = random_selection(cfg, 8)
    ref = (oracle.bwd_gqa if kv_heads else oracle.bwd)(s, q, k, v, dout, idx)
    got = G.gpu_bwd(cfg, q, k, v, dout, idx)
    for name, x, r in zip(("dq", "dk", "dv"), got, ref):
        tol = 1e-4 * np.abs(r).max() if dtype == "fp32" else 1e-2 * max(1.0, np.abs(r).max())
        err = np.abs(x - r).max()
        assert err <= tol, f"{name}: max error {err} > {tol}"
    again = G.gpu_bwd(cfg, q, k, v, dout, idx)
    assert all(np.array_equal(x, y) for x, y in zip(got, again))


# row wavefronts of dK/dV up to which four groups and two share a list (the backward's rule)
SPLIT_LIMITS = {("bf16", 32): (2048, 4096), ("bf16", 64): (2048, 4096), ("bf16", 128): (512, 1024),
                ("fp32", 32): (1408, 8192), ("fp32", 64): (1408, 8192), ("fp32", 128): (0, 2048)}


@pytest.mark.parametrize("dtype,D", list(SPLIT_LIMITS))
@pytest.mark.parametrize("heads,kv_heads,H,W,bh,bw,n", [
    (1, 1, 32, 30, 8, 6, 9),     # b = 48: row wavefronts in pairs, bf16 one, fp32 two per block
    (2, 1, 44, 15, 11, 3, 9),    # b = 33; 330 rows and more to a list, the last piece not full
    (1, 1, 32, 32, 4, 4, 27),    # b = 16: one row wavefront, in two groups or four
    (1, 1, 40, 40, 10, 10, 7),   # b = 100: bf16 unsplit, four, the last of them 16 rows wide
    (1, 1, 28, 40, 7, 10, 7),    # b = 70: three
    (1, 1, 40, 52, 10, 13, 7),   # b = 130: five; head dim 128 two workgroups of three, one empty
])
def test_general_backward_split(G, oracle, dtype, D, heads, kv_heads, H, W, bh, bw, n):
    """One entry as often as it takes for launches whose lists are walked by four groups of
    wavefronts, by two and by one.  The bounds of test_general_backward against the oracle,
    all copies bitwise equal; the bits of dK tell that the smaller launches did split."""
    cfg = shape_ns(1, heads, H, W, bh, bw, D, n, dtype, kv_heads)
    rng = np.random.default_rng(D + n)
    shape = (1, heads, H * W, D)
    q, dout = (rng.standard_normal(shape).astype(np.float32) for _ in range(2))
    k, v = (rng.standard_normal((1, kv_heads, H * W, D)).astype(np.float32) for _ in range(2))
    if dtype == "bf16":
        q, k, v, dout = (round_to_bf16(x) for x in (q, k, v, dout))
    idx = random_selection(cfg, 3)
    ref = (oracle.bwd_gqa if heads > kv_heads else oracle.bwd)(
        oracle.shape_of(cfg), q, k, v, dout, idx)
    rows = 16 if dtype == "fp32" else 32
    per_entry = kv_heads * cfg.n_blocks * -(-cfg.block_tokens // rows)
    four, two = SPLIT_LIMITS[dtype, D]
    bits = []
    for batch in (1, four // per_entry + 1, two // per_entry + 1):
        cfg.batch = batch
        got = G.gpu_bwd(cfg, *(np.repeat(x, batch, axis=0) for x in (q, k, v, dout, idx)))
        for name, x, r in zip(("dq", "dk", "dv"), got, ref):
            assert (x == x[:1]).all(), (name, batch)
            tol = 1e-4 * np.abs(r).max() if dtype == "fp32" else 1e-2 * max(1.0, np.abs(r).max())
            err = np.abs(x[:1] - r).max()
            assert err <= tol, f"{name}, batch {batch}: max error {err} > {tol}"
        bits.append(got[1][0])
    assert not np.array_equal(bits[0], bits[2]) and not np.array_equal(bits[1], bits[2])


@pytest.mark.parametrize("heads,kv_heads,H,W,bh,bw,n", [
    (4, 1, 40, 64, 2, 2, 9),     # m = 640: 80 words per key block, classes by the whole chip
    (2, 1, 32, 128, 2, 2, 9),    # m = 1,024: 64 words, the last map read by its workgroup
    (1, 0, 41, 50, 1, 2, 9),     # m = 1,025: one block in the second round of the order
])
def test_backward_order_of_popular_blocks(G, oracle, heads, kv_heads, H, W, bh, bw, n):
    """A few key blocks that most query blocks attend to, so that every class of the
    working order has members.  A block that is missing from the order keeps the NaN
    that its gradients are filled with.  Bounds of test_general_backward."""
    cfg = shape_ns(1, heads, H, W, bh, bw, 32, n, "fp32", kv_heads)
    m, rng = cfg.n_blocks, np.random.default_rng(n + heads)
    idx = np.empty((1, heads, m, n), dtype=np.int32)
    for a in range(heads):
        weight = 1.0 / (1.0 + rng.permutation(m))
        for i in range(m):
            w = np.where(np.arange(m) == i, 0.0, weight)
            idx[0, a, i] = rng.choice(m, size=n, replace=False, p=w / w.sum())
    q, dout = (rng.standard_normal((1, heads, H * W, 32)).astype(np.float32) for _ in range(2))
    k, v = (rng.standard_normal((1, kv_heads or heads, H * W, 32)).astype(np.float32)
            for _ in range(2))
    ref = (oracle.bwd_gqa if kv_heads else oracle.bwd)(oracle.shape_of(cfg), q, k, v, dout, idx)
    for name, x, r in zip(("dq", "dk", "dv"), G.gpu_bwd(cfg, q, k, v, dout, idx), ref):
        err = np.abs(x - r).max()
        assert err <= 1e-4 * np.abs(r).max(), f"{name}: max error {err}"


@pytest.mark.parametrize("dtype,H,W,bh,bw,D,n,batch", [
    ("fp32", 32, 32, 8, 8, 32, 3, 16),     # 16 blocks x 4 row wavefronts x 2 groups per slice
    ("bf16", 32, 64, 8, 8, 64, 15, 8),     # 32 x 2 x 4, matrix-core kernels
    ("bf16", 32, 64, 8, 16, 128, 7, 8),    # 16 x 4 x 2, a workgroup of four to a CU
])
def test_backward_without_an_order(G, oracle, dtype, H, W, bh, bw, D, n, batch):
    """2,048 wavefronts of dK/dV, or 1,024 where a CU holds four, take the key blocks as they lie,
    one slice more has them ordered: the same lists, sums and bits (dQ, which knows no order, may be split otherwise
    there).  Bounds of test_general_backward."""
    cfg = shape_ns(1, 1, H, W, bh, bw, D, n, dtype)
    q, k, v = rand_qkv(cfg, 31)
    dout = rand_qkv(cfg, 32)[0]
    if dtype == "bf16":
        q, k, v, dout = (round_to_bf16(x) for x in (q, k, v, dout))
    idx = random_selection(cfg, 33)
    ref = oracle.bwd(oracle.shape_of(cfg), q, k, v, dout, idx)
    grads = []
    for cfg.batch in (batch, batch + 1):
        got = G.gpu_bwd(cfg, *(np.repeat(x, cfg.batch, axis=0) for x in (q, k, v, dout, idx)))
        assert all((x == x[:1]).all() for x in got)
        grads.append([x[0] for x in got])
    for name, x, y, r in zip(("dq", "dk", "dv"), *grads, ref):
        assert name == "dq" or np.array_equal(x, y), name
        assert max(np.abs(x - r[0]).max(), np.abs(y - r[0]).max()) <= (1e-4 if dtype == "fp32" else 1e-2) * np.abs(r).max()


def tokens_of_blocks(cfg):
    """int64 [m, b]: the tokens of every block."""
    i = torch.arange(cfg.n_tokens, device="cuda")
    i = i.view(cfg.grid_h // cfg.block_h, cfg.block_h, cfg.grid_w // cfg.block_w, cfg.block_w)
    return i.permute(0, 2, 1, 3).reshape(cfg.n_blocks, cfg.block_tokens)


def block_by_block(cfg, q, k, v, dout, blocks, i):
    """Attention of query block i of one slice (q [N, D] and so on) over the given blocks in 64
    bits: out, log-sum-exp, dq and the block's share of dk and dv, [len(blocks), b, D] each."""
    tok = tokens_of_blocks(cfg)
    rows, keys = tok[i], tok[blocks].reshape(-1)
    qd, kd, vd, gd = (x.double() for x in (q[rows], k[keys], v[keys], dout[rows]))
    scale = cfg.head_dim ** -0.5
    s = qd @ kd.T * scale
    lse = torch.logsumexp(s, dim=1)
    p = torch.exp(s - lse[:, None])
    out = p @ vd
    ds = p * (gd @ vd.T - (gd * out).sum(1, keepdim=True)) * scale
    shape = (len(blocks), cfg.block_tokens, cfg.head_dim)
    return out, lse, ds @ kd, (ds.T @ qd).reshape(shape), (p.T @ gd).reshape(shape)


def close(name, x, ref, dtype, fp32_tol):
    big = float(ref.abs().max())
    tol = fp32_tol * big if dtype == "fp32" else 1e-2 * max(1.0, big)
    err = float((x.double() - ref).abs().max())
    assert err <= tol, f"{name}: max error {err} > {tol}"


@pytest.mark.parametrize("dtype,H,W,bh,bw,D,heads,kv_heads", [
    ("bf16", 272, 512, 16, 16, 64, 9, 9),     # m = 544: eight runs of 64 blocks and 32 more per slice
    ("bf16", 272, 512, 16, 16, 64, 6, 2),     # runs over three heads, the tail 192 blocks
    ("bf16", 512, 132, 8, 12, 128, 8, 8),     # general kernels, m = 704: runs of 128
    ("bf16", 264, 256, 8, 16, 128, 8, 8),     # m = 528: runs of 128, 8 slices in 33 rounds
    ("bf16", 264, 256, 8, 16, 128, 20, 10),   # two slices more than are dealt whole
    ("fp32", 330, 410, 10, 10, 32, 9, 9),     # m = 1,353
    ("fp32", 330, 410, 10, 10, 32, 6, 3),     # and row chunks, 4,059 blocks of two heads each
])
def test_large_slices_in_runs(G, dtype, H, W, bh, bw, D, heads, kv_heads):
    """Slices of more than 32 MB of keys and values, whose query blocks all XCDs share in runs (and
    the key blocks of what is no multiple of eight slices): every row is written, with the bits
    that a launch of its slice alone gives it (launches of so many rows are not split, whatever
    the number of slices), and some blocks of the first and the last slice against 64 bits."""
    import paper_2604_16429_amd as bsa
    from paper_2604_16429_amd import binding
    element = torch.bfloat16 if dtype == "bf16" else torch.float32
    group = heads // kv_heads
    one = shape_ns(1, group, H, W, bh, bw, D, 3, dtype, 1)
    many = shape_ns(1, heads, H, W, bh, bw, D, 3, dtype, kv_heads)
    gen = torch.Generator(device="cuda").manual_seed(D)
    q, k, v, dout = (torch.randn((1, h, H * W, D), generator=gen, device="cuda").to(element)
                     for h in (heads, kv_heads, kv_heads, heads))
    idx = torch.from_numpy(random_selection(many, 4)).cuda()

    def run(cfg, q, k, v, dout, idx):
        p = G.params_of(cfg)
        out, dq, dk, dv = (torch.full_like(x, float("nan")) for x in (q, q, k, v))
        lse = torch.full(q.shape[:3], float("nan"), device="cuda")
        ws = torch.empty(bsa.mosaic_bsa_workspace_bytes(p, binding.OP_BWD), dtype=torch.uint8,
                         device="cuda")
        bsa.mosaic_bsa_fwd(p, q, k, v, idx, out, lse)
        bsa.mosaic_bsa_bwd(p, q, k, v, out, lse, dout, idx, dq, dk, dv, ws)
        return out, lse, dq, dk, dv

    got = run(many, q, k, v, dout, idx)
    assert all(bool(torch.isfinite(x).all()) for x in got)
    out, lse, dq, dk, dv = got
    tok = tokens_of_blocks(many)
    for u in (0, kv_heads - 1):
        of_q, of_kv = slice(u * group, (u + 1) * group), slice(u, u + 1)
        alone = run(one, *(x[:, s].contiguous() for x, s in
                           ((q, of_q), (k, of_kv), (v, of_kv), (dout, of_q), (idx, of_q))))
        for x, y, s in zip(got, alone, (of_q, of_q, of_q, of_kv, of_kv)):
            assert torch.equal(x[:, s], y)
        for j in (0, many.n_blocks // 2, many.n_blocks - 1):
            sum_k = sum_v = 0.0
            for a in range(u * group, (u + 1) * group):
                connected = torch.nonzero((idx[0, a] == j).any(1)).flatten().tolist() + [j]
                for i in connected:
                    blocks = [i] + idx[0, a, i].tolist()
                    o, l, g_q, g_k, g_v = block_by_block(many, q[0, a], k[0, u], v[0, u], dout[0, a],
                                                         blocks, i)
                    sum_k, sum_v = sum_k + g_k[blocks.index(j)], sum_v + g_v[blocks.index(j)]
                    close("out", out[0, a, tok[i]], o, dtype, 1e-5)
                    close("lse", lse[0, a, tok[i]], l, "fp32", 1e-5 if dtype == "fp32" else 1e-3)
                    close("dq", dq[0, a, tok[i]], g_q, dtype, 1e-4)
            close("dk", dk[0, u, tok[j]], sum_k, dtype, 1e-4)
            close("dv", dv[0, u, tok[j]], sum_v, dtype, 1e-4)


@pytest.mark.parametrize("dtype,H,W,bh,bw,D,heads,kv_heads", [
    ("bf16", 272, 512, 16, 16, 64, 9, 9),
    ("bf16", 272, 512, 16, 16, 64, 4, 2),     # two jobs in runs over two heads
    ("fp32", 330, 410, 10, 10, 32, 9, 9),
])
def test_large_slices_three_branch(G, dtype, H, W, bh, bw, D, heads, kv_heads):
    """The same for the three branches, forward and backward: both attention branches of a launch
    in runs, the local branch's key blocks as well."""
    import paper_2604_16429_amd as bsa
    element = torch.bfloat16 if dtype == "bf16" else torch.float32
    group, lh, lw, n = heads // kv_heads, 1, 2 if W // bw % 2 == 0 else 1, 3
    one = shape_ns(1, group, H, W, bh, bw, D, n, dtype, 1)
    many = shape_ns(1, heads, H, W, bh, bw, D, n, dtype, kv_heads)
    gen = torch.Generator(device="cuda").manual_seed(D + 1)
    q, k, v, dout = (torch.randn((1, h, H * W, D), generator=gen, device="cuda").to(element)
                     for h in (heads, kv_heads, kv_heads, heads))
    gates = torch.rand((1, heads, H * W, 3), generator=gen, device="cuda")

    def run(cfg, q, k, v, gates, dout):
        p = G.params_of(cfg)
        out, dq, dk, dv, dgates = (torch.full_like(x, float("nan")) for x in (q, q, k, v, gates))
        idx = torch.empty((1, cfg.heads, cfg.n_blocks, n), dtype=torch.int32, device="cuda")
        ws, ws_b = (torch.empty(size(p, lh, lw), dtype=torch.uint8, device="cuda") for size in (
            bsa.mosaic_bsa_three_branch_workspace_bytes,
            bsa.mosaic_bsa_three_branch_bwd_workspace_bytes))
        bsa.mosaic_bsa_fwd_three_branch(p, lh, lw, q, k, v, gates, out, idx, ws)
        bsa.mosaic_bsa_bwd_three_branch(p, lh, lw, q, k, v, gates, dout, idx, ws, dq, dk, dv,
                                        dgates, ws_b)
        return idx, out, dq, dk, dv, dgates

    got = run(many, q, k, v, gates, dout)
    idx, out = got[:2]
    assert all(bool(torch.isfinite(x).all()) for x in got[1:])
    tok = tokens_of_blocks(many)
    for u in (0, kv_heads - 1):
        of_q, of_kv = slice(u * group, (u + 1) * group), slice(u, u + 1)
        alone = run(one, *(x[:, s].contiguous() for x, s in
                           ((q, of_q), (k, of_kv), (v, of_kv), (gates, of_q), (dout, of_q))))
        for x, y, s in zip(got, alone, (of_q, of_q, of_q, of_kv, of_kv, of_q)):
            assert torch.equal(x[:, s], y)
        kbar, vbar = (x[0, u][tok].double().mean(1) for x in (k, v))
        for a in range(u * group, (u + 1) * group):
            for i in (0, many.n_blocks // 3, many.n_blocks - 1):
                w = torch.softmax(kbar @ q[0, a, tok[i]].double().mean(0) * D ** -0.5, dim=0)
                fg = block_by_block(many, q[0, a], k[0, u], v[0, u], dout[0, a], idx[0, a, i].tolist(), i)
                local = block_by_block(many, q[0, a], k[0, u], v[0, u], dout[0, a],
                                       [i // lw * lw + x for x in range(lw)], i)
                parts = torch.stack([(w @ vbar).expand_as(fg[0]), fg[0], local[0]], dim=2)
                ref = (parts * gates[0, a, tok[i]].double()[:, None]).sum(2)
                close("out", out[0, a, tok[i]], ref, dtype, 1e-5)
                close("dgates", got[5][0, a, tok[i]],
                      (parts * dout[0, a, tok[i]].double()[:, :, None]).sum(1), dtype, 1e-4)


@pytest.mark.parametrize("D", [64, 128])
def test_backward_fp32_score_rounding(G, oracle, D):
    """Scores whose terms all have one sign, mean s (22 and 31 here): a chain of c
    products is rounded by 2^-24 / sqrt(3) sqrt(c / 3) of its value, so that a score in
    four chains of D / 4 is off by about 2^-24 0.6 (sqrt(D / 12) / 2 + 1) s, 1.25 to 1.5
    times 2^-24 s, and in one chain of D by 2.7 to 3.8 times (less what it shares with
    the lse).  The error of a score is the relative error of its weight in dK and dV:
    2-norm within 1.8 times 2^-24 s."""
    cfg = shape_ns(1, 2, 32, 32, 8, 4, D, 2, "fp32")
    rng = np.random.default_rng(1)
    q, k = (rng.uniform(0.5, 1.5, size=(1, 2, 1024, D)).astype(np.float32)
            * np.float32(0.7 * np.sqrt(512 / D)) for _ in range(2))
    v, dout = (rng.standard_normal((1, 2, 1024, D)).astype(np.float32) for _ in range(2))
    idx = random_selection(cfg, 1)
    score = (q[0, 0] @ k[0, 0].T).mean() / np.sqrt(D)
    _, dk, dv = G.gpu_bwd(cfg, q, k, v, dout, idx)
    _, rk, rv = oracle.bwd(oracle.shape_of(cfg), q, k, v, dout, idx)
    for name, x, r in (("dk", dk, rk), ("dv", dv, rv)):
        err = np.linalg.norm(x - r) / np.linalg.norm(r)
        assert err <= 1.8 * 2.0 ** -24 * score, f"{name}: {err / score * 2 ** 24}"


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_backward_list_of_connected_blocks_full(G, oracle, dtype):
    """Blocks of one token and 2,112 query blocks that all attend to block 0: its list
    is filled to its end and walked to the last of the entries that repeat the last
    block, then filled again.  Bounds of test_general_backward, relative to the sum
    that 2,112 terms make."""
    cfg = shape_ns(1, 1, 33, 64, 1, 1, 32, 1, dtype)
    q, k, v = inputs_of(cfg, 1)
    dout = inputs_of(cfg, 2)[0]
    idx = np.zeros((1, 1, cfg.n_blocks, 1), dtype=np.int32)
    idx[0, 0, 0] = 1
    ref = oracle.bwd(oracle.shape_of(cfg), q, k, v, dout, idx)
    for name, x, r in zip(("dq", "dk", "dv"), G.gpu_bwd(cfg, q, k, v, dout, idx), ref):
        err = np.abs(x - r).max()
        assert err <= (1e-4 if dtype == "fp32" else 1e-2) * max(1.0, np.abs(r).max()), (name, err)


@pytest.mark.parametrize("dtype,H,W,bh,bw,D,kv_heads", [
    ("fp32", 10, 20, 5, 5, 64, 1),      # general kernels
    ("bf16", 32, 40, 16, 20, 32, 2),    # two workgroups per block
    ("bf16", 32, 64, 8, 8, 64, 1),      # head dim 64
    ("bf16", 32, 64, 8, 16, 128, 2),    # head dim 128
    ("bf16", 32, 64, 16, 16, 128, 1),
])
def test_backward_in_place(G, dtype, H, W, bh, bw, D, kv_heads):
    """Gradients over inputs: dq in the memory of out (the order of the key blocks,
    which lies in dq, must not be there before out is read), dk and dv in those of k
    and v.  Bitwise the result of separate tensors."""
    import paper_2604_16429_amd as bsa
    from paper_2604_16429_amd import binding
    cfg = shape_ns(2, 2, H, W, bh, bw, D, 3, dtype, kv_heads)
    p = G.params_of(cfg)
    element = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(D)
    q, dout = (torch.randn((2, 2, H * W, D), generator=gen, device="cuda").to(element)
               for _ in range(2))
    k, v = (torch.randn((2, kv_heads, H * W, D), generator=gen, device="cuda").to(element)
            for _ in range(2))
    idx = G.select_dev(cfg, q, k)
    out, lse = G.fwd_dev(cfg, q, k, v, idx)
    ws = torch.empty(bsa.mosaic_bsa_workspace_bytes(p, binding.OP_BWD), dtype=torch.uint8,
                     device="cuda")
    ref = [torch.empty_like(t) for t in (q, k, v)]
    bsa.mosaic_bsa_bwd(p, q, k, v, out, lse, dout, idx, *ref, ws)

    o = out.clone()
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    bsa.mosaic_bsa_bwd(p, q, k, v, o, lse, dout, idx, o, dk, dv, ws)
    assert all(torch.equal(x, r) for x, r in zip((o, dk, dv), ref))
    o, k2, v2 = out.clone(), k.clone(), v.clone()
    bsa.mosaic_bsa_bwd(p, q, k2, v2, o, lse, dout, idx, o, k2, v2, ws)
    assert all(torch.equal(x, r) for x, r in zip((o, k2, v2), ref))


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("heads,kv_heads,H,W,bh,bw,D,n,lh,lw", [
    (2, 0, 9, 11, 1, 1, 32, 4, 3, 1),      # b = 1: parts of a tile without a token; m = 99
    (2, 1, 10, 13, 5, 1, 128, 3, 2, 13),   # b = 5, m = 26: a column tile with idle columns
    (4, 1, 33, 22, 3, 11, 64, 5, 11, 1),   # b = 33, m = 22, wide rows, group of 4
    (2, 2, 24, 36, 4, 9, 32, 2, 1, 2),     # b = 36, m = 24
    (1, 0, 66, 2, 2, 2, 64, 3, 1, 1),      # m = 33: one column past a 32-column tile
])
def test_general_three_branch(G, oracle, dtype, heads, kv_heads, H, W, bh, bw, D, n, lh, lw):
    """Both directions of the three-branch form where the token parts of the branch
    gradients, the 32-column tiles of the coarse branch's backward and the general
    attention kernels have remainders.  Bounds of the repository's three-branch
    tests: fp32 1e-4, bf16 2e-2 of max(1, largest entry); outputs 1e-5 / 2e-2."""
    cfg = shape_ns(1, heads, H, W, bh, bw, D, n, dtype, kv_heads=kv_heads)
    rng = np.random.default_rng(60 + H + W + D)
    q, dout = (rng.standard_normal((1, heads, H * W, D)).astype(np.float32) for _ in range(2))
    k, v = (rng.standard_normal((1, kv_heads or heads, H * W, D)).astype(np.float32)
            for _ in range(2))
    if dtype == "bf16":
        q, k, v, dout = (round_to_bf16(x) for x in (q, k, v, dout))
    gates = rng.uniform(-1.0, 1.0, size=(1, heads, H * W, 3)).astype(np.float32)
    s = oracle.shape_of(cfg, own_is_candidate=True)
    out, sel, dq, dk, dv, dg = G.gpu_three_branch_fwd_bwd(cfg, q, k, v, gates, dout, lh, lw)
    assert np.array_equal(sel, oracle.select_all(s, q, oracle.expand_kv(k, heads)))
    rq, rk, rv, rg, value = oracle.bwd_three_branch(s, q, k, v, gates, dout, sel, lh, lw)
    tol = 2e-2 if dtype == "bf16" else 1e-4
    for name, x, r in zip(("dq", "dk", "dv", "dgates"), (dq, dk, dv, dg), (rq, rk, rv, rg)):
        err = np.abs(x - r).max()
        assert err <= tol * max(1.0, np.abs(r).max()), f"{name}: {err}"
    ref = np.asarray(value)
    assert np.abs(out - ref).max() <= (2e-2 if dtype == "bf16" else 1e-5 * np.abs(ref).max())


@pytest.mark.parametrize("heads,H,W,D", [
    (1, 64, 128, 64),        # m = 2,048: ranking and coarse branch in one launch
    (1, 128, 128, 32),       # m = 4,096: in two, for the ranking's place on the CU
    (1, 160, 160, 32),       # m = 6,400: in one again, neither fits twice
])
def test_three_branch_many_blocks(G, oracle, heads, H, W, D):
    """Both ways to launch the ranking and the coarse branch, tiles of 2 x 2."""
    cfg = shape_ns(1, heads, H, W, 2, 2, D, 5, "fp32")
    q, k, v = rand_qkv(cfg, H + D)
    gates = np.random.default_rng(D).uniform(0.0, 1.0, size=(1, heads, H * W, 3)).astype(np.float32)
    s = oracle.shape_of(cfg, own_is_candidate=True)
    ref, sel_ref, _ = oracle.fwd_three_branch(s, q, k, v, gates, 2, 2)
    got, sel = G.gpu_fwd_three_branch(cfg, q, k, v, gates, 2, 2)
    assert np.array_equal(sel, sel_ref)
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("H,W,bh,bw,n,levels", [
    (24, 36, 2, 2, 70, 0),       # m = 216, more picks than one round of 32 places
    (48, 48, 2, 2, 100, 0),      # m = 576: two key blocks per thread, four rounds
    (48, 48, 2, 2, 16, 2),       # few distinct scores: more than 64 reach the threshold
    (24, 36, 2, 2, 215, 2),      # n = m - 1 with ties
    (5, 26, 1, 2, 64, 3),        # m = 65: a lane whose only candidate is removed
    (1, 128, 1, 64, 1, 0),       # m = 2
    (48, 48, 2, 2, 100, 1),      # all scores equal
    (48, 48, 2, 2, 100, -1),     # clustered: distinct, equal in the threshold's first bits
    (24, 36, 2, 2, 215, -1),
    (48, 96, 2, 2, 90, -2),      # clustered on top of a few that stand out
])
def test_selection_rounds(G, oracle, H, W, bh, bw, n, levels):
    """Top-n in rounds of a threshold: exact indices whatever the scores look like.
    levels > 0: keys and queries take that many small integer values per block, so
    that scores are exact and mostly equal; < 0: they share a large mean, so that
    scores are clustered (-2: some key blocks are larger by half)."""
    cfg = shape_ns(2, 2, H, W, bh, bw, 32, min(n, (H // bh) * (W // bw) - 1), "fp32")
    q, k, _ = rand_qkv(cfg, 31 + n)
    if levels < 0:
        q, k = q + np.float32(100.0), np.float32(0.01) * k + np.float32(100.0)
        if levels == -2:
            k[:, :, :3 * W] *= np.float32(1.5)
    if levels > 0:
        rng = np.random.default_rng(n)
        rows, cols = H // bh, W // bw
        for x in (q, k):
            v = rng.integers(0, levels, size=(2, 2, rows, 1, cols, 1, 1)).astype(np.float32)
            x[:] = np.broadcast_to(v, (2, 2, rows, bh, cols, bw, 32)).reshape(x.shape)
    s = oracle.shape_of(cfg)
    assert np.array_equal(G.gpu_select(cfg, q, k), oracle.select(s, q, k))


def many_blocks(cfg, kind, seed):
    """q, k of tiles of 2 x 2 whose scores are random, mostly equal, rising with the block
    index, falling, or subnormal."""
    rng = np.random.default_rng(seed)
    shape = (cfg.batch, cfg.heads, cfg.n_tokens, cfg.head_dim)
    q, k = (rng.standard_normal(shape).astype(np.float32) for _ in range(2))
    if kind == "levels":
        rows, cols = cfg.grid_h // 2, cfg.grid_w // 2
        for x in (q, k):
            v = rng.integers(0, 2, size=shape[:2] + (rows, 1, cols, 1, 1)).astype(np.float32)
            x[:] = np.broadcast_to(v, shape[:2] + (rows, 2, cols, 2, shape[3])).reshape(shape)
    elif kind in ("rising", "falling"):
        q = 1.0 + 0.01 * q
        ramp = np.arange(cfg.n_tokens, dtype=np.float32) / cfg.n_tokens
        k = 0.001 * k + (ramp if kind == "rising" else -ramp)[None, None, :, None]
    elif kind == "subnormal":
        q, k = q * np.float32(1e-20), k * np.float32(3e-21)
    return q.astype(np.float32), k.astype(np.float32)


@pytest.mark.parametrize("kind", ["random", "levels", "rising", "falling", "subnormal"])
@pytest.mark.parametrize("heads,H,W,D,n", [
    (10, 26, 122, 128, 32),     # 793 blocks: 25 in the last group of 64 and of 32 rows
    (10, 32, 96, 128, 1),       # 768: three whole steps
    (10, 64, 96, 64, 8),        # 1,536: the smallest at head dim 64
    (10, 58, 106, 64, 17),      # 1,537: one block in the last group
    (10, 14, 878, 32, 16),      # 3,073
])
def test_selection_many_blocks(G, oracle, kind, heads, H, W, D, n):
    """Rankings of many blocks on the matrix cores: exact indices."""
    cfg = shape_ns(1, heads, H, W, 2, 2, D, n, "fp32")
    assert cfg.n_blocks * D >= 98304 and heads * -(-cfg.n_blocks // 32) * D >= 30000
    q, k = many_blocks(cfg, kind, H + n)
    assert np.array_equal(G.gpu_select(cfg, q, k), oracle.select(oracle.shape_of(cfg), q, k))


def test_selection_many_blocks_grouped_heads_and_own_block(G, oracle):
    """The same with three query heads to a key head, and with the own block a candidate."""
    cfg = shape_ns(1, 9, 26, 122, 2, 2, 128, 5, "fp32", kv_heads=3)
    q, k = many_blocks(cfg, "random", 1)
    k = k[:, :3].copy()
    assert np.array_equal(G.gpu_select(cfg, q, k), oracle.select_gqa(oracle.shape_of(cfg), q, k))
    cfg = shape_ns(1, 10, 26, 122, 2, 2, 128, 5, "fp32")
    q, k = many_blocks(cfg, "random", 2)
    gates = np.ones((1, 10, cfg.n_tokens, 3), dtype=np.float32)
    ref = oracle.select_all(oracle.shape_of(cfg, own_is_candidate=True), q, k)
    assert np.array_equal(G.gpu_fwd_three_branch(cfg, q, k, k, gates, 1, 1)[1], ref)


def test_selection_many_blocks_of_nan(G):
    """Scores that are no numbers still give distinct blocks other than the own one."""
    cfg = shape_ns(1, 10, 26, 122, 2, 2, 128, 7, "fp32")
    q, k = many_blocks(cfg, "random", 3)
    q[0, 3] = np.nan
    k[0, 4, :2000] = np.nan
    k[0, 5, 100] = np.nan
    idx = np.sort(G.gpu_select(cfg, q, k), axis=-1)
    own = np.arange(cfg.n_blocks)[:, None]
    assert idx.min() >= 0 and idx.max() < cfg.n_blocks and (idx[0] != own).all()
    assert (np.diff(idx, axis=-1) > 0).all()


@pytest.mark.parametrize("batch", [1 << 18, 1 << 20])
def test_general_more_than_2_32_work_items(G, batch):
    """2^22 and 2^24 slices of one token: with 1,024 and 256 threads per slice kernels
    would need 2^32 work items, which one launch cannot have.
    The output is v and the only weight 1, so dv = dout and dq = dk = 0 up to the fp32
    sums of dP and delta (32 terms each, at most 2^-19 of sum |dO v|, times scale and
    key, which are below 1)."""
    import paper_2604_16429_amd as bsa
    from paper_2604_16429_amd import binding
    heads, D = 16, 32
    p = bsa.Params(batch, heads, 1, 1, 1, 1, D, 0, binding.BF16)
    gen = torch.Generator(device="cuda").manual_seed(9)
    q, k, v, dout = (torch.rand((batch, heads, 1, D), generator=gen, device="cuda",
                                dtype=torch.bfloat16) for _ in range(4))
    out, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.empty((batch, heads, 1), device="cuda")
    ws = torch.empty(bsa.mosaic_bsa_workspace_bytes(p, binding.OP_BWD), dtype=torch.uint8,
                     device="cuda")
    none = torch.empty((batch, heads, 1, 0), dtype=torch.int32, device="cuda")
    bsa.mosaic_bsa_fwd(p, q, k, v, none, out, lse)
    bsa.mosaic_bsa_bwd(p, q, k, v, out, lse, dout, none, dq, dk, dv, ws)
    assert torch.equal(out, v)
    assert (dv.float() - dout.float()).abs().max() <= 2.0 ** -8
    for x in (dq, dk):
        assert x.float().abs().max() <= 32 * 2.0 ** -19


def test_general_backward_more_than_2_32_work_items(G):
    """2^25 blocks of 17 tokens, two to a slice that both attend to all of it, 128 work items
    each in dQ: more than one launch can have.  One buffer of 68 GiB serves as q, out and
    dout, lse is 3.  Against the formulas in 64 bits for the first batch entries and the
    last, which take another launch; bound of test_general_backward."""
    import paper_2604_16429_amd as bsa
    from paper_2604_16429_amd import binding
    batch, heads, N, D = 1 << 18, 64, 34, 32
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 180 << 30:
        pytest.skip("needs 180 GiB of device memory")
    p = bsa.Params(batch, heads, N, 1, 17, 1, D, 1, binding.F32, 0.0, 1)
    gen = torch.Generator(device="cuda").manual_seed(10)
    some = torch.randn((1021, N, D), generator=gen, device="cuda")      # q, repeated
    q = torch.empty((batch, heads, N, D), device="cuda")
    rows = q.view(-1, N, D)
    for at in range(0, rows.shape[0], 1021 << 10):
        part = rows[at:at + (1021 << 10)]
        part.copy_(some.repeat(-(-part.shape[0] // 1021), 1, 1)[:part.shape[0]])
    k, v = (torch.randn((batch, 1, N, D), generator=gen, device="cuda") for _ in range(2))
    lse = torch.full((batch, heads, N), 3.0, device="cuda")
    idx = torch.tensor([1, 0], dtype=torch.int32, device="cuda").repeat(batch * heads)
    dq = torch.full_like(q, float("nan"))
    dk, dv = (torch.full_like(k, float("nan")) for _ in range(2))
    ws = torch.empty(bsa.mosaic_bsa_workspace_bytes(p, binding.OP_BWD), dtype=torch.uint8,
                     device="cuda")
    bsa.mosaic_bsa_bwd(p, q, k, v, q, lse, q, idx, dq, dk, dv, ws)
    assert not any(torch.isnan(x.sum()) for x in (dq, dk, dv))
    for e in (0, 1, batch - 2, batch - 1):
        qe, ke, ve = (x[e].double() for x in (q, k, v))
        w = torch.exp(qe @ ke[0].T / D ** 0.5 - 3.0)
        ds = w * (qe @ ve[0].T - (qe * qe).sum(-1, keepdim=True)) / D ** 0.5
        for name, x, r in (("dq", dq, ds @ ke[0]), ("dk", dk, (ds.transpose(1, 2) @ qe).sum(0)),
                           ("dv", dv, (w.transpose(1, 2) @ qe).sum(0))):
            err = (x[e].double() - r).abs().max()
            assert err <= 1e-4 * r.abs().max(), f"{name} of entry {e}: {err}"


@pytest.mark.parametrize("dtype,H,W,D,grouped", [
    ("fp32", 2048, 2064, 128, False), ("fp32", 1024, 2064, 128, True),
    ("bf16", 4096, 4128, 64, False), ("bf16", 4096, 4128, 32, True),
])
def test_general_rows_past_32_bit_offsets(G, dtype, H, W, D, grouped):
    """A slice (or the query slices that share a key/value slice) of more than 2 GiB
    takes 64-bit addresses.  Block i attends to itself and to its successor, so the
    last blocks' outputs and gradients follow from three blocks: checked there against
    float64 reverse mode (fp32: outputs 1e-5, gradients 1e-4 of the largest entry;
    bf16: the bounds of the two tests of the general kernels)."""
    import paper_2604_16429_amd as bsa
    from paper_2604_16429_amd import binding
    bh, bw, heads = 16, 43, 2 if grouped else 1
    bf16 = dtype == "bf16"
    p = bsa.Params(1, heads, H, W, bh, bw, D, 1, binding.BF16 if bf16 else binding.F32, 0.0, 1)
    element = torch.bfloat16 if bf16 else torch.float32
    assert heads * H * W * D * element.itemsize > 1 << 31
    N, m, rows = H * W, (H // bh) * (W // bw), W // bw
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, dout = (torch.randn((1, heads, N, D), generator=gen, device="cuda", dtype=element)
               for _ in range(2))
    k, v = (torch.randn((1, 1, N, D), generator=gen, device="cuda", dtype=element)
            for _ in range(2))
    idx = ((torch.arange(m, device="cuda", dtype=torch.int32) + 1) % m).view(1, 1, m, 1)
    idx = idx.expand(1, heads, m, 1).contiguous()
    out, dq = torch.empty_like(q), torch.empty_like(q)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    lse = torch.empty((1, heads, N), device="cuda")
    ws = torch.empty(bsa.mosaic_bsa_workspace_bytes(p, binding.OP_BWD), dtype=torch.uint8,
                     device="cuda")
    bsa.mosaic_bsa_fwd(p, q, k, v, idx, out, lse)
    bsa.mosaic_bsa_bwd(p, q, k, v, out, lse, dout, idx, dq, dk, dv, ws)

    def block(x, i):                      # [heads, b, D] in float64
        x = x[0].view(x.shape[1], H // bh, bh, rows, bw, D)
        return x[:, i // rows, :, i % rows].reshape(x.shape[0], bh * bw, D).double()

    j = m - 2                             # attended by blocks m - 3 and m - 2
    kv = {i: (block(k, i).requires_grad_(), block(v, i).requires_grad_()) for i in range(m - 3, m)}
    qs = {i: block(q, i).requires_grad_() for i in (m - 3, m - 2)}
    total = 0.0
    for i, x in qs.items():
        keys, values = (torch.cat([kv[i][t], kv[i + 1][t]], dim=1) for t in (0, 1))
        o = torch.softmax(x @ keys.transpose(1, 2) / D ** 0.5, dim=-1) @ values
        err = (block(out, i) - o).abs()
        bound = 2.0 ** -8 * o.abs() + 2.0 ** -14 * 6 if bf16 else 1e-5 * o.abs().max()
        assert (err <= bound).all(), f"out of block {i}: {err.max()}"
        total = total + (o * block(dout, i)).sum()
    total.backward()
    for name, x, r in (("dq", block(dq, j), qs[j].grad), ("dk", block(dk, j), kv[j][0].grad),
                       ("dv", block(dv, j), kv[j][1].grad)):
        err = (x - r).abs().max()
        top = r.abs().max().item()
        assert err <= (1e-2 * max(1.0, top) if bf16 else 1e-4 * top), f"{name} of block {j}: {err}"


@pytest.mark.parametrize("H,W,bh,bw,D,n,lh,lw", [
    (32, 64, 8, 8, 64, 6, 2, 2),         # the kernels specialised for head dim 64
    (32, 64, 8, 16, 128, 6, 2, 2),       # for head dim 128
    (20, 60, 10, 10, 32, 6, 2, 2),       # the general ones
])
def test_three_branch_upstream_rounding_cancels(G, H, W, bh, bw, D, n, lh, lw):
    """Equal values everywhere: every branch returns that value whatever its weights
    are, so dq = 0.  The gated upstream gradients are rounded to bf16 (2^-9 of every
    entry); dP and delta have to be taken from the same rounded values, or the
    rounding's dot product with v, about 2^-9 / 3 |g dO| sqrt(D) per token, weighs
    the mean key into dq.  Bound: the fp32 sums of dP and delta, D 2^-24 sum |dO v|
    each, in the two attention branches, times the softmax scale and the largest
    key; gates are at most 1."""
    cfg = shape_ns(1, 2, H, W, bh, bw, D, n, "bf16")
    rng = np.random.default_rng(17 + D)
    q, k, dout = (rng.standard_normal((1, 2, H * W, D)).astype(np.float32) for _ in range(3))
    q, k, dout = (round_to_bf16(x) for x in (q, k + 2.0, dout))
    v = np.broadcast_to(rng.choice([-1.0, 1.0], size=(1, 2, 1, D)), q.shape).astype(np.float32)
    gates = rng.uniform(0.0, 1.0, size=(1, 2, H * W, 3)).astype(np.float32)
    dq = G.gpu_three_branch_fwd_bwd(cfg, q, k, np.ascontiguousarray(v), gates, dout, lh, lw)[2]
    per_sum = D * 2.0 ** -24 * np.abs(dout).sum(axis=-1).max()
    assert np.abs(dq).max() <= 2 * 2 * per_sum * np.abs(k).max() / np.sqrt(D)
