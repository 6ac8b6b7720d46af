"""Linear layers (and the fp32 attention) at the row counts where their plan changes kernel, tile or
division of the contraction axis: the dense block (QKV routed into the cache, O with fp32 output, FC1 with GELU, FC2)
against the oracle."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import TOL, GpuBlock, oracle_dense, rel_err, to_dev, to_np  # noqa: E402


@pytest.mark.parametrize("dtype,B,M,d,H,F", [
    ("f32", 1, 1, 64, 1, 64),     # one row, fewer k-steps than wavefronts, fewer key tiles than wavefronts
    ("f32", 1, 17, 128, 1, 192),  # row remainder 1 of a 32-row tile, head_dim 128
    ("f32", 3, 11, 1024, 16, 4096),   # 33 rows of three samples in one 64-row tile, divided contraction
    ("f32", 2, 129, 512, 8, 1088),    # row remainders, an MLP width that is no power of two
    ("bf16", 1, 1, 64, 1, 64),            # one row, two k-steps: most wavefronts of a workgroup get none
    ("bf16", 1, 7, 1024, 16, 4096),       # 16-row tiles without staging
    ("bf16", 3, 6, 1024, 8, 4096),        # 18 rows of three samples: a tile spans samples, 32 features a workgroup
    ("bf16", 1, 33, 960, 15, 1984),       # row remainder 1, width not a power of two
    ("bf16", 1, 64, 2048, 16, 8192),      # FC2 divided seven ways (32 k-tiles do not divide evenly)
    ("bf16", 2, 65, 1024, 16, 4096),      # 130 rows: 128x64 tiles divided eight ways, 64x64 undivided
    ("bf16", 1, 257, 1024, 16, 4096),     # first row count without the unstaged kernel: 64x128 tiles
    ("bf16", 1, 257, 128, 2, 256),        # 64x64 tiles, contraction of two k-tiles on a ring of three
    ("bf16", 1, 700, 1024, 16, 4096),     # 128x128 tiles (ring of four), divided and not
    ("bf16", 4, 225, 1920, 30, 7680),     # 192x128 tiles, K/V rows routed across samples inside a tile
    ("bf16", 2, 924, 1920, 15, 7680),     # 256x192 tiles, ragged rows and columns
    ("bf16", 2, 1300, 64, 1, 6144),       # many tiles, a single k-tile
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
