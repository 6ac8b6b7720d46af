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
    (1, 130, 3559, 256, 4, 8),      # 58 tiles in ranges of 8; the last of 2, one for each group
    (1, 130, 3495, 256, 4, 8),      # 57 tiles: in the last range the first group has none
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


@pytest.mark.parametrize("B,n,Lp,d,H,ways,dead", [
    (1, 40, 100, 128, 2, 101, 64),          # one group, undivided: the first tile
    (1, 40, 100, 256, 2, 101, 70),          # head_dim 128, and six keys of the next
    (1, 20, 4000, 1024, 8, 108, 512),       # one group, ranges of 8 tiles: the whole first range
    (10, 150, 441, 512, 4, 201, 64),        # two groups: the first group's first tile
    (10, 150, 441, 512, 4, 201, 320),       # all five tiles of the first group
    (8, 100, 441, 1024, 16, 201, 256),      # head_dim 64, the same with four
    (1, 130, 3495, 256, 4, 208, 512),       # two groups, ranges: the whole first range
])
def test_keys_whose_scores_overflow_to_minus_infinity_weigh_nothing(B, n, Lp, d, H, ways, dead):
    """The first `dead` keys of the cache have a score of -inf, all others of 0: the attention is the mean of the other
    values, also where a tile, a group's share or a range holds no finite score.  The weights are 0 and 1, so in fp32
    only the sum over V is rounded; the attention is rounded to bf16 once, the block's output once more."""
    Dh, L, bf = d // H, Lp + n, True
    assert fv.load_library()["_ZN4fvar14attention_waysEiiiii"](B, n, L, H, Dh) == ways
    x = wl.activations_lowrank(B, n, d, seed=90 + n, bf16=bf)
    Kp, Vp = wl.kv_prefix(B, Lp, H, Dh, seed=91, bf16=bf)
    Kp = np.zeros_like(Kp)
    Kp[:, :dead, :, 0] = -1e30
    w = {"w_qkv": np.zeros((3 * d, d)), "b_qkv": np.zeros(3 * d), "w_o": np.eye(d), "w_fc1": np.zeros((d, d)),
         "w_fc2": np.zeros((d, d))}
    w = {k: v.astype(np.float32) for k, v in w.items()}
    w["b_qkv"][:d:Dh] = 1e30
    blk = GpuBlock(d, H, d, "bf16", w, wl.round_to_bf16(Kp), Vp, L)
    y = to_np(blk.dense(to_dev(x, "bf16"))).astype(np.float64)
    att = Vp[:, dead:].astype(np.float64).sum(axis=1).reshape(B, 1, d) / (L - dead)      # the block's own keys add 0
    expect = x.astype(np.float64) + att
    within = bool(np.all(np.abs(y - expect) <= 2.0 ** -8 * (np.abs(att) + np.abs(expect)) + 1e-6))
    assert within
