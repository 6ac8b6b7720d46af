"""Attention whose keys are divided between two wavefront groups of a workgroup: tile counts that do and do not
divide evenly, a last tile of one key, query remainders, both head sizes and key ranges on top, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2512_16483_amd as fv
import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import TOL, GpuBlock, oracle_dense, rel_err, to_dev, to_np  # noqa: E402


@pytest.mark.parametrize("B,n,Lp,d,H,ranges", [
    (20, 33, 441, 512, 4, 1),       # 8 tiles, one active wavefront and one query in the next
    (10, 150, 441, 512, 4, 1),      # 10 tiles
    (11, 200, 441, 512, 4, 1),      # 11 tiles, the last with one key
    (5, 256, 441, 1024, 16, 1),     # head_dim 64, 256 queries per workgroup, 11 tiles
    (8, 100, 441, 1024, 16, 1),     # head_dim 64, 128 queries per workgroup, 9 tiles
    (1, 300, 300, 256, 4, 1),       # query remainder 44, 10 tiles
    (12, 20, 917, 1024, 8, 2),      # 15 tiles in ranges of 8, each for two groups; the last of 7
    (1, 20, 4629, 256, 4, 8),       # head_dim 64, 73 tiles in ranges of 10; the last of 3
])
def test_two_wavefront_groups_share_the_keys(B, n, Lp, d, H, ranges):
    ways = fv.load_library()["_ZN4fvar14attention_waysEiiiii"]
    assert ways(B, n, Lp + n, H, d // H) == 200 + ranges
    F, tol = 2 * d, TOL["bf16"]
    x = wl.activations_lowrank(B, n, d, seed=80 + n, bf16=True)
    w = wl.block_weights(d, F, seed=81, bf16=True, std=0.8 / np.sqrt(d))
    Kp, Vp = wl.kv_prefix(B, Lp, H, d // H, seed=82, bf16=True)
    yo, Kn, Vn = oracle_dense(x, w, H, Kp, Vp)
    blk = GpuBlock(d, H, F, "bf16", w, Kp, Vp, Lp + n + 5)
    blk.K[:, Lp + n:], blk.V[:, Lp + n:] = float("nan"), float("nan")     # rows past the cache's end are not read
    y = blk.dense(to_dev(x, "bf16"))
    torch.cuda.synchronize()
    assert rel_err(to_np(blk.K[:, Lp:Lp + n]), Kn) <= tol
    assert rel_err(to_np(blk.V[:, Lp:Lp + n]), Vn) <= tol
    assert rel_err(to_np(y), yo) <= tol
