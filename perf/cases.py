"""The work that a user of this package has it do, as cases that can be timed.

A case is one attention call (or one training pass of it) on a grid, through
the package's public entry points:

  op "fwd"     mosaic_bsa_select + mosaic_bsa_fwd (inference with one softmax)
  op "train"   the same, then mosaic_bsa_bwd
  op "fwd3"    mosaic_bsa_fwd_three_branch (the paper's output form)
  op "train3"  the same, then mosaic_bsa_bwd_three_branch

Sizes are in the terms of mosaic_bsa_params; kv_heads = heads unless grouped
query attention is used.  `local_h`, `local_w` (three-branch form): tiles per
large local block.  `ensemble`: the batch entries are members that share a base
field and differ by small perturbations (else they are independent fields).
"""
from __future__ import annotations

import math

import torch

import paper_2604_16429_amd as bsa
from paper_2604_16429_amd import binding


def _case(name, op, dtype, batch, heads, kv_heads, grid_h, grid_w, block_h, block_w, head_dim,
          n_select, local_h=0, local_w=0, ensemble=False, corr_len=6.0):
    c = dict(op=op, dtype=dtype, batch=batch, heads=heads, kv_heads=kv_heads, grid_h=grid_h,
             grid_w=grid_w, block_h=block_h, block_w=block_w, head_dim=head_dim,
             n_select=n_select, local_h=local_h, local_w=local_w, ensemble=ensemble,
             corr_len=corr_len)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a test-sized grid in fp32, all launches and latency.
        _case("tiny_fp32_fwd", "fwd", "fp32", 1, 2, 2, 32, 64, 8, 8, 32, 4, corr_len=4.0),
        # One forecast member on the 1.5 degree grid: few slices, the chip half idle.
        _case("grid15_single_fwd", "fwd", "bf16", 1, 8, 8, 120, 240, 8, 8, 64, 8),
        # One attention layer of a 24-member ensemble step on the 1.5 degree grid.
        _case("grid15_ensemble_fwd", "fwd", "bf16", 24, 16, 16, 120, 240, 8, 8, 64, 16,
              ensemble=True),
        # The 0.25 degree grid: one million tokens, 4,050 blocks of 256 tokens.
        _case("grid025_fwd", "fwd", "bf16", 1, 16, 16, 720, 1440, 16, 16, 64, 16, corr_len=24.0),
        # Length scaling at head dim 32, batch 1, 16 heads: 131,072 tokens in
        # consecutive blocks of 128.
        _case("length_d32_fwd", "fwd", "bf16", 1, 16, 16, 1024, 128, 1, 128, 32, 16),
        # Training pass of the 1.5 degree grid at head dim 128.
        _case("grid15_d128_train", "train", "bf16", 4, 16, 16, 120, 240, 8, 16, 128, 12),
        # Fine-tuning on the ensemble with grouped heads (4 query heads per key/value head).
        _case("grid15_grouped_train", "train", "bf16", 12, 16, 4, 120, 240, 8, 8, 64, 16,
              ensemble=True),
        # Tiles that are no power of two: 10 x 10 divides the 1.5 degree grid as well.
        _case("ragged_tile_train", "train", "bf16", 2, 8, 8, 120, 240, 10, 10, 64, 8),
        # Full precision training pass (gradient checks, small studies).
        _case("grid15_fp32_train", "train", "fp32", 1, 8, 8, 120, 240, 8, 8, 64, 8),
        # The paper's first stage (49,152 pixels, 24 blocks) as its ensemble forecast runs it.
        _case("stage1_fwd3", "fwd3", "bf16", 24, 12, 3, 384, 128, 1, 128, 64, 24, 8, 1,
              ensemble=True),
        # The paper's second stage (12,288 pixels, 12 blocks), a training pass.
        _case("stage2_train3", "train3", "bf16", 8, 16, 4, 96, 128, 1, 128, 64, 12, 8, 1),
        # The paper's bottleneck (3,072 pixels, 4 blocks) for one member: latency.
        _case("bottleneck_fwd3", "fwd3", "bf16", 1, 20, 5, 24, 128, 1, 128, 64, 4, 8, 1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Tiles of the configurations: 64, 128 and 256 tokens, widths a power of two.
_TILES = [(8, 8), (8, 16), (16, 16), (1, 128), (4, 32), (16, 8), (1, 64)]


def draw(rng):
    """One more case: any entry point, type, head dim, tile and grid that the
    listed ones stand for, at most as much work as the largest of them (fp32 and
    tiles that are no power of two: at most 4e11 flop)."""
    while True:
        op = rng.choice(["fwd", "fwd", "train", "fwd3", "train3"])
        dtype = "fp32" if rng.random() < 0.2 else "bf16"
        head_dim = rng.choice([32, 64, 64, 128])
        plain = rng.random() < 0.6
        if plain:
            bh, bw = rng.choice(_TILES)
        else:
            bh, bw = rng.randint(3, 16), rng.randint(3, 20)
            if not 32 <= bh * bw <= 256:
                continue
        lh, lw = (0, 0)
        if op.endswith("3"):
            lh, lw = rng.choice([(8, 1), (3, 3), (2, 2), (2, 1), (1, 1)])
        # grid of tiles: m log-uniform, wider than high for 2-D tiles
        m = _log_int(rng, 16, 4096)
        if bh == 1:
            rows, cols = m, 1
        else:
            rows = max(2, int(round(math.sqrt(m * bw / bh / 2.0))))
            cols = max(2, int(round(m / rows)))
        if lh:
            rows, cols = max(1, rows // lh) * lh, max(1, cols // lw) * lw if bh > 1 else 1
            if bh == 1:
                lw = 1
        m = rows * cols
        if not 8 <= m <= 4096:
            continue
        kv = rng.randint(1, 8)
        group = rng.choice([1, 1, 2, 4])
        c = _case(None, op, dtype, _log_int(rng, 1, 24), kv * group, kv, rows * bh, cols * bw, bh,
                  bw, head_dim, min(_log_int(rng, 2, 32), m - 1), lh, lw,
                  ensemble=rng.random() < 0.5)
        w = work(c)
        slow = dtype == "fp32" or not plain or head_dim == 32
        if w["flops"] <= (4e11 if slow else 1.4e13) and w["bytes"] <= 1.0e10:
            return c


def _params(c):
    return bsa.Params(c["batch"], c["heads"], c["grid_h"], c["grid_w"], c["block_h"],
                      c["block_w"], c["head_dim"], c["n_select"],
                      binding.BF16 if c["dtype"] == "bf16" else binding.F32, 0.0,
                      c["kv_heads"])


def _smoothing(n, corr_len, periodic, device):
    """[n, n] Gaussian smoothing along one axis, reflecting or periodic."""
    i = torch.arange(n, device=device, dtype=torch.float32)
    d = i[:, None] - i[None, :]
    s = torch.zeros(n, n, device=device)
    for shift in (-1, 0, 1):
        if periodic:
            s += torch.exp(-0.5 * ((d + shift * n) / corr_len) ** 2)
        else:
            e = d if shift == 0 else i[:, None] + i[None, :] + 1 - (shift + 1) * n
            s += torch.exp(-0.5 * (e / corr_len) ** 2)
    return s


def _field(gen, c, heads, lat, lon):
    """Smooth unit-variance fields plus 0.1 white noise, fp32 [heads, N, D]."""
    H, W, D = c["grid_h"], c["grid_w"], c["head_dim"]
    ch = heads * D
    x = torch.randn(H, W * ch, generator=gen, device="cuda")
    x = lat @ x
    x = x.view(H, W, ch).transpose(0, 1).reshape(W, H * ch)
    x = lon @ x
    x = x.view(W, H, heads, D).permute(2, 1, 0, 3).reshape(heads, H * W, D)
    x /= x.square().mean(dim=1, keepdim=True).sqrt()
    x += 0.1 * torch.randn(x.shape, generator=gen, device="cuda")
    return x


def _tensor(gen, c, heads, lat, lon):
    """[B, heads, N, D] in the case's element type."""
    dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    shape = (c["batch"], heads, c["grid_h"] * c["grid_w"], c["head_dim"])
    out = torch.empty(shape, dtype=dtype, device="cuda")
    base = None
    for e in range(c["batch"]):
        if c["ensemble"]:
            if base is None:
                base = _field(gen, c, heads, lat, lon)
            out[e] = base + 0.05 * torch.randn(base.shape, generator=gen, device="cuda")
        else:
            out[e] = _field(gen, c, heads, lat, lon)
    return out


def prepare(case, seed):
    c = dict(case)
    p = _params(c)
    lat = _smoothing(c["grid_h"], c["corr_len"], False, "cuda")
    lon = _smoothing(c["grid_w"], c["corr_len"], True, "cuda")
    gens = [torch.Generator(device="cuda").manual_seed(seed * 8 + t) for t in range(5)]
    s = {"op": c["op"], "p": p, "local": (c["local_h"], c["local_w"])}
    s["q"] = _tensor(gens[0], c, c["heads"], lat, lon)
    s["k"] = _tensor(gens[1], c, c["kv_heads"], lat, lon)
    s["v"] = _tensor(gens[2], c, c["kv_heads"], lat, lon)
    s["out"] = torch.empty_like(s["q"])
    s["idx"] = torch.empty((p.batch, p.heads, p.n_blocks, p.n_select), dtype=torch.int32,
                           device="cuda")
    rows = (p.batch, p.heads, p.n_tokens)
    if c["op"] in ("train", "train3"):
        s["dout"] = torch.randn(s["q"].shape, generator=gens[3],
                                device="cuda").to(s["q"].dtype)
        s["dq"], s["dk"], s["dv"] = (torch.empty_like(s[t]) for t in ("q", "k", "v"))

    def space(n):
        return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")

    if c["op"] in ("fwd", "train"):
        s["lse"] = torch.empty(rows, dtype=torch.float32, device="cuda")
        s["ws"] = space(bsa.mosaic_bsa_workspace_bytes(p, binding.OP_SELECT))
        if c["op"] == "train":
            s["ws_b"] = space(bsa.mosaic_bsa_workspace_bytes(p, binding.OP_BWD))
    else:
        s["gates"] = torch.rand(rows + (3,), generator=gens[4], device="cuda")
        s["ws"] = space(bsa.mosaic_bsa_three_branch_workspace_bytes(p, *s["local"]))
        if c["op"] == "train3":
            s["dgates"] = torch.empty_like(s["gates"])
            s["ws_b"] = space(bsa.mosaic_bsa_three_branch_bwd_workspace_bytes(p, *s["local"]))
    return s


def run(s):
    p, op = s["p"], s["op"]
    if op in ("fwd", "train"):
        bsa.mosaic_bsa_select(p, s["q"], s["k"], s["idx"], s["ws"])
        bsa.mosaic_bsa_fwd(p, s["q"], s["k"], s["v"], s["idx"], s["out"], s["lse"])
        if op == "fwd":
            return s["idx"], s["out"], s["lse"]
        bsa.mosaic_bsa_bwd(p, s["q"], s["k"], s["v"], s["out"], s["lse"], s["dout"], s["idx"],
                           s["dq"], s["dk"], s["dv"], s["ws_b"])
        return s["idx"], s["out"], s["lse"], s["dq"], s["dk"], s["dv"]
    lh, lw = s["local"]
    bsa.mosaic_bsa_fwd_three_branch(p, lh, lw, s["q"], s["k"], s["v"], s["gates"], s["out"],
                                    s["idx"], s["ws"])
    if op == "fwd3":
        return s["idx"], s["out"]
    bsa.mosaic_bsa_bwd_three_branch(p, lh, lw, s["q"], s["k"], s["v"], s["gates"], s["dout"],
                                    s["idx"], s["ws"], s["dq"], s["dk"], s["dv"], s["dgates"],
                                    s["ws_b"])
    return s["idx"], s["out"], s["dq"], s["dk"], s["dv"], s["dgates"]


def work(case):
    c = case
    esz = 2 if c["dtype"] == "bf16" else 4
    B, h, kvh, D = c["batch"], c["heads"], c["kv_heads"], c["head_dim"]
    N, b = c["grid_h"] * c["grid_w"], c["block_h"] * c["block_w"]
    m, n = N // b, c["n_select"]
    three, train = c["op"].endswith("3"), c["op"].startswith("train")
    q_bytes, kv_bytes = B * h * N * D * esz, B * kvh * N * D * esz
    rows = B * h * N
    # q, k, v in; out and the selection out; lse out, or gates in
    nbytes = 2 * q_bytes + 2 * kv_bytes + 4 * B * h * m * n + (12 if three else 4) * rows
    attended = (n + c["local_h"] * c["local_w"]) if three else n + 1
    attention = 4.0 * B * h * N * attended * b * D
    blocks = 2.0 * B * h * m * m * D                     # pooled scores
    flops = attention + blocks * (2 if three else 1)     # coarse branch: weights x values
    if train:
        # dout in; dq, dk, dv (and the gate gradients) out; five products for two
        nbytes += 2 * q_bytes + 2 * kv_bytes + (12 * rows if three else 0)
        flops += 2.5 * attention + (8.0 * B * h * m * m * D if three else 0.0)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    """Selected indices are exact (differ 0).  Floating outputs: about four times
    the distance to a double-precision evaluation of the same definition, which
    is at most 2.1e-6 / 4.1e-5 (rel / max) in fp32 and 3.2e-3 / 4.6e-2 in bf16
    over the listed cases at a reduced batch (gradients; forward outputs less)."""
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 3e-4, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.2, "differ": 0.0}
