"""Linear layers (and the fp32 attention) at the row counts where their plan changes kernel, tile or
division of the contraction axis: the dense block (QKV routed into the cache, O with fp32 output, FC1 with GELU, FC2)
against the oracle.  That the rows below get the plans they are here for is checked without a GPU, in
test_abi_host.py."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import TOL, GpuBlock, oracle_dense, rel_err, to_dev, to_np  # noqa: E402


@pytest.mark.parametrize("dtype,B,M,d,H,F", [
    ("f32", 1, 1, 64, 1, 64),     # one row, fewer k-steps than wavefronts, fewer key tiles than wavefronts
    ("f32", 1, 17, 128, 1, 192),  # row remainder 1 of a 32-row tile, head_dim 128
    ("f32", 3, 11, 1024, 16, 4096),   # 33 rows of three samples
    ("f32", 2, 129, 512, 8, 1088),    # row remainders, an MLP width that is no power of two
    ("bf16", 1, 1, 64, 1, 64),            # one row, two k-steps: most wavefronts of a workgroup get none
    ("bf16", 1, 7, 1024, 16, 4096),       # 16x16 by rings per wavefront
    ("bf16", 3, 6, 1024, 8, 4096),        # 18 rows of three samples: a tile spans samples, 32 rows a workgroup
    ("bf16", 1, 33, 960, 15, 1984),       # row remainder 1, width not a power of two
    ("bf16", 1, 64, 2048, 16, 8192),      # rings of 48x32, 16x32 and 32x64, FC2 in four shares
    ("bf16", 2, 65, 1024, 16, 4096),      # 130 rows: rings of 48x64, 32x32 and 64x64, undivided
    ("bf16", 1, 257, 1024, 16, 4096),     # first row count without rings: 64x64, 128x64, 64x128 in six shares
    ("bf16", 1, 257, 128, 2, 256),        # 64x64 tiles, contraction of two k-tiles on a ring of three
    ("bf16", 1, 700, 1024, 16, 4096),     # 128x128 tiles (ring of four), divided and not
    ("bf16", 4, 225, 1920, 30, 7680),     # 192x128 tiles, K/V rows routed across samples inside a tile
    ("bf16", 2, 924, 1920, 15, 7680),     # 256x192 tiles, ragged rows and columns
    ("bf16", 2, 1300, 64, 1, 6144),       # many tiles, a single k-tile
    ("bf16", 3, 12, 2048, 16, 8192),      # 36 rows of three samples in one 32-row tile and the next
    ("bf16", 4, 36, 4096, 32, 1024),      # QKV divided in two: 192x128 tiles over four samples
    ("bf16", 3, 214, 4096, 32, 64),       # QKV with a last round divided eight ways, tiles across samples
    ("bf16", 2, 805, 4096, 32, 64),       # the same in three, 256x256 tiles
    ("bf16", 1, 64, 512, 8, 5440),        # FC2: 85 steps for eight wavefronts
    ("bf16", 3, 25, 3072, 48, 64),        # QKV divided in three: 128x128 tiles over three samples
])
def test_linear_layers_across_plans(dtype, B, M, d, H, F):
    Lp, bf, tol = 5, dtype == "bf16", TOL[dtype]
    x = wl.activations_lowrank(B, M, d, seed=700 + M, bf16=bf)
    w = wl.block_weights(d, F, seed=701, bf16=bf, std=0.8 / np.sqrt(d), with_bias=True, with_affine=True)
    Kp, Vp = wl.kv_prefix(B, Lp, H, d // H, seed=702, bf16=bf)
    yo, Kn, Vn = oracle_dense(x, w, H, Kp, Vp)
    blk = GpuBlock(d, H, F, dtype, w, Kp, Vp, Lp + M + 3)
    blk.K[:, Lp + M:], blk.V[:, Lp + M:] = 7.0, 7.0
    y = blk.dense(to_dev(x, dtype))
    torch.cuda.synchronize()
    assert rel_err(to_np(blk.K[:, Lp:Lp + M]), Kn) <= tol
    assert rel_err(to_np(blk.V[:, Lp:Lp + M]), Vn) <= tol
    assert rel_err(to_np(y), yo) <= tol
    assert np.array_equal(to_np(blk.K[:, :Lp]), Kp) and bool((blk.K[:, Lp + M:] == 7.0).all())
    assert np.array_equal(to_np(blk.V[:, :Lp]), Vp) and bool((blk.V[:, Lp + M:] == 7.0).all())


@pytest.mark.parametrize("B,M,d,H,F", [
    (3, 90, 1088, 17, 1088),      # QKV: 64x64 by four groups, 17 k-tiles: the last trip is one group's alone; K/V rows routed across samples
    (1, 65, 1088, 17, 1088),      # rings, 17 steps for eight wavefronts
    (1, 520, 960, 15, 2240),      # FC2: 64x64 by four groups, 35 k-tiles: one group has none in the last trip
    (1, 257, 512, 8, 1088),       # FC2: row remainder 1
    (1, 330, 1088, 17, 4096),     # FC1 (GELU): 128x64 by two groups, 17 k-tiles
    (1, 400, 960, 15, 4160),      # FC2: the same divided four ways, 17 and 14 k-tiles a workgroup
    (3, 100, 2048, 16, 2112),     # QKV: 64x128 by two groups, K/V rows routed across samples inside a tile
])
def test_linear_layers_by_wavefront_groups(B, M, d, H, F):
    """The tiles whose k-tiles are dealt to groups of wavefronts: counts that do not divide evenly."""
    test_linear_layers_across_plans("bf16", B, M, d, H, F)


@pytest.mark.parametrize("d,rows", [
    (256, 5), (256, 200),                 # rings per wavefront
    (1024, 40), (1024, 969), (1024, 970), (1024, 1152), (1024, 1153), (1024, 1537), (1024, 2048),
    (1024, 12289), (1920, 6145), (2048, 2050),
])
def test_second_mlp_layer_rounds_once(d, rows):
    """y = residual + product, both fp32 until the one rounding to bf16, whichever tile, division or
    merge the plan picks.  Constructed so that nothing before that rounding is inexact: attention and
    its projection are 0 (h = x), the hidden layer is gelu(16) = 16 everywhere, and a row of W_fc2
    holds two entries whose products are a value of 8 bits and one 2^-9 .. 2^-14 of it, so the fp32
    product is exact in every order of summation but does not fit bf16.  Exact equality: the expected
    value is one fp32 addition, rounded once."""
    F, H = 4 * d, d // 64
    rng = np.random.default_rng(rows)
    x = wl.round_to_bf16(rng.standard_normal((1, rows, d)).astype(np.float32) * 2)
    hi = wl.round_to_bf16(rng.standard_normal(d).astype(np.float32))
    lo = wl.round_to_bf16(hi * rng.uniform(2.0 ** -14, 2.0 ** -9, d).astype(np.float32))
    w = {"w_qkv": np.zeros((3 * d, d)), "w_o": np.zeros((d, d)), "w_fc1": np.zeros((F, d)),
         "b_fc1": np.full(F, 16.0), "w_fc2": np.zeros((d, F))}
    w = {n: v.astype(np.float32) for n, v in w.items()}
    w["w_fc2"][np.arange(d), rng.integers(0, F // 2, d)] = hi / 16
    w["w_fc2"][np.arange(d), rng.integers(F // 2, F, d)] = lo / 16
    Kp = np.zeros((1, 3, H, 64), np.float32)
    blk = GpuBlock(d, H, F, "bf16", w, Kp, Kp, 3 + rows)
    y = blk.dense(to_dev(x, "bf16")).cpu()
    expect = (torch.from_numpy(x) + torch.from_numpy(hi + lo)).to(torch.bfloat16)
    assert np.array_equal((hi.astype(np.float64) + lo).astype(np.float32), hi + lo)
    assert torch.equal(y, expect), f"{(y != expect).sum().item()} of {y.numel()} differ"


@pytest.mark.parametrize("dtype,B,M,d,H,F", [
    ("f32", 3, 6, 1024, 8, 4096),         # 16x32, 16x16 and 16x32 in four shares; 18 rows of three samples
    ("f32", 5, 50, 320, 5, 1280),         # 250 rows: remainder 10; ten contraction steps for eight wavefronts
    ("f32", 1, 85, 960, 15, 3840),        # 48x32 in four shares; row remainder 5
    ("f32", 1, 200, 1024, 16, 4096),      # 48x64 (QKV), 32x32, 64x64
    ("f32", 1, 3, 2048, 32, 64),          # FC1: 16x16 in eight shares
    ("f32", 1, 33, 768, 12, 5440),        # FC2: 48x32 in eight shares, 170 steps for 64 wavefronts
    ("f32", 1, 57, 1088, 17, 5440),       # FC2: 32x32 in two shares
    ("bf16", 1, 43, 1536, 24, 6144),      # FC2: 48x32 in four shares, row remainder 11
    ("bf16", 1, 99, 1536, 24, 6144),      # FC2: 48x64 in four shares, second row tile of 35 rows
    ("bf16", 1, 141, 4096, 32, 1024),     # FC2: 64x64
    ("bf16", 7, 14, 1024, 16, 4096),      # 98 rows of seven samples: K/V rows routed across samples; 48x32, 16x32, 32x64
    ("bf16", 1, 48, 1920, 30, 7680),      # 48x32, 16x32, 32x64, FC2 in four shares
    ("bf16", 1, 33, 1920, 30, 7680),      # FC2: 64x64 in eight shares
    ("bf16", 1, 3, 768, 12, 8192),        # FC2: 32x16 in eight shares
    ("bf16", 3, 8, 4096, 32, 16384),      # FC2: 32x32 in two shares; 24 rows of three samples
])
def test_linear_layers_with_a_ring_per_wavefront(dtype, B, M, d, H, F):
    """The kernel of a few rows (fp32: of all), each of its instances, with row remainders and shares."""
    test_linear_layers_across_plans(dtype, B, M, d, H, F)


@pytest.mark.parametrize("B,M,d,H,F", [
    (1, 436, 768, 12, 3072),      # FC2: 64x64 in three shares
    (4, 100, 512, 8, 2048),       # FC2: 64x64 in four shares, tiles over four samples
    (1, 72, 1920, 30, 7680),      # FC2: 128x64 in eight shares, row remainder 72
    (1, 180, 1536, 24, 5440),     # FC2: 64x128 in seven shares, 85 k-tiles, row remainder 52
    (1, 137, 1536, 24, 6144),     # FC2: 64x128 in seven shares, row remainder 9
])
def test_small_tiles_that_still_divide_the_contraction(B, M, d, H, F):
    """Where the kernel of a few rows is not the faster one, small tiles in shares run as before."""
    test_linear_layers_across_plans("bf16", B, M, d, H, F)
