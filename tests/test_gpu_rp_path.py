"""GPU parity of the random-projection input path and of the on-GPU factor construction: the HIP
kernels through the C ABI against the CPU oracle on the same seeded inputs.

Bars as for the main path: copies and index work bit-exact; bf16 outputs within 2e-2, fp32
outputs within 1e-4, measured as max_i |g_i - o_i| / max(|o_i|, rms(o))."""
import numpy as np
import pytest
import torch

import oracle
from oracle import factors, rp_path
import paper_2512_16483_amd as fv
import workloads as wl

pytestmark = pytest.mark.gpu

from gpu_util import TOL, GpuBlock, rel_err, tdtype, to_dev, to_np  # noqa: E402


def _ctx(d, dtype, H=None):
    H = H or d // 64
    return fv.Context(hidden=d, heads=H, head_dim=d // H, ffn_hidden=4 * d, dtype=dtype)


def _q(B, M, r, seed, dtype, per_sample):
    """Q = z / sqrt(r) in the storage type, [B or 1, M, r]."""
    z = wl.normal_draws(B if per_sample else 1, M, r, seed=seed)
    Q = (z / np.sqrt(float(r))).astype(np.float32)
    return wl.round_to_bf16(Q) if dtype == "bf16" else Q


def _qt_dev(Q, dtype):
    return to_dev(np.ascontiguousarray(np.swapaxes(Q, 1, 2)), dtype)      # [B or 1, r, M]


# ----------------------------------------------------------------------------- projection
@pytest.mark.parametrize("dtype,B,M,rows,d,per_sample", [
    ("bf16", 2, 72, 5, 128, False),          # one full chunk of 64 tokens + a ragged one
    ("bf16", 3, 200, 130, 192, True),        # two row tiles, ragged rows, ragged column tile
    ("bf16", 1, 576, 231, 1920, False),      # scale 24 of the depth-30 model
    ("bf16", 2, 1024, 64, 256, True),
    ("bf16", 1, 8, 1, 64, False),            # minimal
    ("f32", 2, 36, 7, 64, True),
    ("f32", 1, 256, 32, 1024, False),        # the fp32 configuration
])
def test_rp_project_parity(dtype, B, M, rows, d, per_sample):
    x = wl.activations_lowrank(B, M, d, seed=50 + M, bf16=dtype == "bf16")
    Q = _q(B, M, rows, 60 + M, dtype, per_sample)
    ctx = _ctx(d, dtype)
    out = torch.full((B, rows, d), float("nan"), dtype=tdtype(dtype), device="cuda")
    fv.fvar_rp_project(ctx, _qt_dev(Q, dtype), per_sample, to_dev(x, dtype), B, M, rows, out)
    torch.cuda.synchronize()
    got = to_np(out)
    for b in range(B):
        ref = rp_path.rp_input(Q[b if per_sample else 0], x[b], bf16=dtype == "bf16")
        assert rel_err(got[b], ref) <= TOL[dtype], (b, rel_err(got[b], ref))


@pytest.mark.parametrize("B,M,rows,d,per_sample", [
    (12, 128, 128, 4096, False),     # 128x256 tiles, two k-tiles on a three-stage ring
    (12, 64, 64, 4096, True),        # a single k-tile, Q per sample
    (24, 320, 320, 2048, True),      # rows of one and a quarter 256-row tiles
    (16, 256, 250, 3136, False),     # 256x256 tiles, ragged rows and columns
    (16, 192, 192, 3072, True),      # 192x256 tiles, three k-tiles
    (32, 512, 500, 384, False),      # 256x128 tiles, ragged rows
    (3, 1024, 700, 4096, True),      # long contraction, several rounds of workgroups
])
def test_rp_project_tiled_path(B, M, rows, d, per_sample):
    """Shapes on whole 64-token k-tiles with enough output tiles to fill the chip run on the tiled
    MFMA kernel of the linear layers with the token map as a k-major operand: every tile
    configuration it can pick, against the oracle on every sample."""
    x = wl.activations_lowrank(B, M, d, seed=150 + M + rows, bf16=True)
    Q = _q(B, M, rows, 160 + M + rows, "bf16", per_sample)
    ctx = _ctx(d, "bf16")
    out = torch.full((B, rows, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    fv.fvar_rp_project(ctx, _qt_dev(Q, "bf16"), per_sample, to_dev(x, "bf16"), B, M, rows, out)
    torch.cuda.synchronize()
    got = to_np(out)
    assert np.isfinite(got).all()
    for b in range(B):
        ref = rp_path.rp_input(Q[b if per_sample else 0], x[b], bf16=True)
        assert rel_err(got[b], ref) <= TOL["bf16"], (b, rel_err(got[b], ref))


@pytest.mark.parametrize("B,M,rows,d,per_sample", [
    (2, 56, 50, 192, True),          # less than one k-tile
    (1, 2312, 692, 2048, False),     # 64x128 tiles by two groups, one chunk past the last whole k-tile
    (1, 520, 60, 256, False),        # 64x128 by two groups, nine k-tiles: the last trip is one group's alone
    (24, 584, 50, 1024, True),       # 64x128 by one group: every workgroup reads a strip of its own
    (5, 136, 130, 1024, False),      # the samples share Q: its rows end inside the last k-tile
    (4, 440, 190, 4096, True),       # 128x128 tiles, seven of the eight chunks
    (4, 840, 330, 4096, True),       # 192x128
    (3, 1000, 700, 4096, True),      # 192x256
    (16, 264, 250, 3136, False),     # 256x256
    (32, 520, 500, 384, False),      # 128x256
])
def test_rp_project_ragged_token_counts(B, M, rows, d, per_sample):
    """Token counts that are no multiple of the 64-token k-tile.  What lies behind a sample's map and
    behind Q must not matter, not even as NaN: each sample is run among neighbours of NaN."""
    x = wl.activations_lowrank(B, M, d, seed=250 + M + rows, bf16=True)
    Q = _q(B, M, rows, 260 + M + rows, "bf16", per_sample)
    ctx = _ctx(d, "bf16")
    xd, qd, nan = to_dev(x, "bf16"), _qt_dev(Q, "bf16"), float("nan")
    q_room = torch.full((qd.numel() + 64 * M,), nan, dtype=torch.bfloat16, device="cuda")
    q_room[:qd.numel()] = qd.flatten()
    for b in range(B) if B < 8 else (0, B // 2, B - 1):
        room = torch.full((B + 1, M, d), nan, dtype=torch.bfloat16, device="cuda")
        room[b] = xd[b]
        out = torch.zeros((B, rows, d), dtype=torch.bfloat16, device="cuda")
        fv.fvar_rp_project(ctx, q_room, per_sample, room, B, M, rows, out)
        torch.cuda.synchronize()
        ref = rp_path.rp_input(Q[b if per_sample else 0], x[b], bf16=True)
        assert rel_err(to_np(out[b]), ref) <= TOL["bf16"], b
        assert bool(torch.isnan(out[:b]).all()) and bool(torch.isnan(out[b + 1:]).all())


def test_rp_project_rows_beyond_32bit_offsets():
    """Token counts whose 64 rows of Q^T span 4 GiB: the rows are taken a few at a time.  A selection matrix gives
    rows of the map bit for bit; one past the last row of a tile and the last token are among them."""
    M, rows, d = (1 << 26) + 8, 37, 64
    x = torch.empty((1, M, d), dtype=torch.bfloat16, device="cuda").normal_(generator=torch.Generator("cuda").manual_seed(1))
    q = torch.zeros((rows, M), dtype=torch.bfloat16, device="cuda")
    idx = torch.tensor([(M - 1) * (rows - 1 - t) // (rows - 1) for t in range(rows)])     # the last token first
    assert int(idx.min()) == 0 and int(idx.max()) == M - 1
    q[torch.arange(rows), idx] = 1.0
    out = torch.full((1, rows, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    fv.fvar_rp_project(_ctx(d, "bf16"), q, False, x, 1, M, rows, out)
    torch.cuda.synchronize()
    assert torch.equal(out[0], x[0, idx])


def test_rp_project_tiled_path_selection_matrix_bitexact():
    # products with 1 and 0 are exact: a column-selection Q reproduces the rows bit for bit
    B, M, rows, d = 12, 128, 128, 4096
    x = wl.activations_iid(B, M, d, seed=171, bf16=True)
    rng = np.random.default_rng(6)
    Q = np.zeros((B, M, rows), np.float32)
    idx = np.stack([rng.permutation(M)[:rows] for _ in range(B)])
    for b in range(B):
        Q[b, idx[b], np.arange(rows)] = 1.0
    ctx = _ctx(d, "bf16")
    out = torch.empty((B, rows, d), dtype=torch.bfloat16, device="cuda")
    fv.fvar_rp_project(ctx, _qt_dev(Q, "bf16"), True, to_dev(x, "bf16"), B, M, rows, out)
    torch.cuda.synchronize()
    for b in range(B):
        assert np.array_equal(to_np(out[b]), x[b][idx[b]])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rp_project_with_selection_matrix_is_the_gather(dtype):
    # products with 1 and 0 are exact, so a column-selection Q must reproduce the rows bit for bit
    B, M, rows, d = 2, 136, 40, 192
    x = wl.activations_iid(B, M, d, seed=71, bf16=dtype == "bf16")
    rng = np.random.default_rng(5)
    Q = np.zeros((B, M, rows), np.float32)
    idx = np.stack([np.sort(rng.choice(M, rows, replace=False)) for _ in range(B)])
    for b in range(B):
        Q[b, idx[b], np.arange(rows)] = 1.0
    ctx = _ctx(d, dtype)
    out = torch.empty((B, rows, d), dtype=tdtype(dtype), device="cuda")
    fv.fvar_rp_project(ctx, _qt_dev(Q, dtype), True, to_dev(x, dtype), B, M, rows, out)
    torch.cuda.synchronize()
    for b in range(B):
        assert np.array_equal(to_np(out[b]), x[b][idx[b]])


# ----------------------------------------------------------------------------- raw-cache fill
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,M,k,d", [(2, 37, 11, 128), (1, 64, 0, 64), (3, 50, 50, 192), (2, 576, 231, 1920)])
def test_cache_fill_bitexact(dtype, B, M, k, d):
    bf = dtype == "bf16"
    Cm = wl.activations_iid(B, M, d, seed=81, bf16=bf)
    yk = wl.activations_iid(B, max(k, 1), d, seed=82, bf16=bf)[:, :k]
    rng = np.random.default_rng(M + k)
    keep = np.stack([np.sort(rng.choice(M, k, replace=False)) for _ in range(B)]).astype(np.int32).reshape(B, k)
    drop = np.stack([np.setdiff1d(np.arange(M), keep[b]) for b in range(B)]).astype(np.int32).reshape(B, M - k)
    ctx = _ctx(d, dtype)
    kd, dd = torch.from_numpy(keep).cuda(), torch.from_numpy(drop).cuda()
    ykd, Cd = to_dev(yk, dtype), to_dev(Cm, dtype)
    y = torch.full((B, M, d), float("nan"), dtype=tdtype(dtype), device="cuda")
    fv.fvar_cache_fill(ctx, ykd if k else None, kd if k else None, dd if k < M else None, B, M, k,
                       Cd if k < M else None, y)
    # in place: the cache buffer itself receives the kept rows
    Cin = Cd.clone()
    fv.fvar_cache_fill(ctx, ykd if k else None, kd if k else None, dd if k < M else None, B, M, k,
                       Cin, Cin)
    torch.cuda.synchronize()
    for b in range(B):
        ref = rp_path.cache_fill(yk[b], keep[b], Cm[b])
        assert np.array_equal(to_np(y[b]), ref)
        assert np.array_equal(to_np(Cin[b]), ref)


# ----------------------------------------------------------------------------- factors
@pytest.mark.parametrize("dtype,B,M,d,r,rank,noise,per_sample", [
    ("bf16", 2, 72, 128, 8, 24, 0.1, True),
    ("bf16", 1, 200, 192, 40, 60, 0.1, False),       # r not a multiple of 32, ragged row block
    ("bf16", 2, 576, 1920, 64, 102, 0.1, False),     # depth-30 geometry, scale 24
    ("bf16", 1, 256, 256, 128, 200, 0.1, False),     # largest rank
    ("bf16", 1, 64, 64, 16, 16, 0.0, False),         # exactly rank r: lossless
    ("f32", 2, 36, 64, 8, 12, 0.1, True),
    ("f32", 1, 256, 1024, 32, 32, 0.05, False),      # the fp32 configuration
])
def test_cache_factors_parity(dtype, B, M, d, r, rank, noise, per_sample):
    bf = dtype == "bf16"
    Cm = wl.cached_feature(B, M, d, rank, seed=90 + M, noise=noise)
    if bf:
        Cm = wl.round_to_bf16(Cm)
    Q = _q(B, M, r, 91 + M, dtype, per_sample)
    ctx = _ctx(d, dtype)
    Cd = to_dev(Cm, dtype)
    w_c = torch.full((B, M, r), float("nan"), dtype=tdtype(dtype), device="cuda")
    g_c = torch.full((B, r, d), float("nan"), dtype=tdtype(dtype), device="cuda")
    ws = torch.empty(fv.fvar_factors_workspace_bytes(ctx, B, M, r), dtype=torch.uint8, device="cuda")
    fv.fvar_cache_factors(ctx, Cd, _qt_dev(Q, dtype), per_sample, B, M, r, 0.0, w_c, g_c, ws)
    torch.cuda.synchronize()
    Wg, Gg = to_np(w_c), to_np(g_c)
    for b in range(B):
        Wo, Go = factors.stored_factors(Cm[b], Q[b if per_sample else 0], bf16=bf)
        assert rel_err(Gg[b], Go) <= TOL[dtype], ("G", b, rel_err(Gg[b], Go))
        assert rel_err(Wg[b], Wo) <= TOL[dtype], ("W", b, rel_err(Wg[b], Wo))
        # the restoration the factors exist for: as close to C as the oracle's
        C64 = Cm[b].astype(np.float64)
        res_g = np.linalg.norm(Wg[b].astype(np.float64) @ Gg[b].astype(np.float64) - C64)
        res_o = np.linalg.norm(Wo.astype(np.float64) @ Go.astype(np.float64) - C64)
        assert res_g <= res_o * 1.02 + (4e-3 if bf else 1e-6) * np.linalg.norm(C64)
        if noise == 0.0:       # rank r exactly (up to the bf16 rounding of C, W and G themselves)
            assert res_g <= (2e-2 if bf else 1e-5) * np.linalg.norm(C64)


@pytest.mark.parametrize("B,M,d,r,ridge", [
    (1, 520, 512, 16, 0.0),       # one 16-wide pivot block, three empty tiles
    (2, 264, 256, 56, 1e-10),     # partly padded last block of four
    (1, 328, 1024, 72, 1e-10),    # five of eight blocks
    (1, 4096, 4096, 128, 0.0),    # every block, 64 k-tiles
    (3, 1000, 320, 104, 1e-10),   # ragged rows and token chunks
    (1, 1024, 4096, 64, 0.0),     # T in two shares, 128 x 64 tiles
    (1, 264, 4096, 32, 1e-10),    # T in three shares, 64 x 64 tiles
    (1, 520, 4096, 8, 0.0),       # T in four
    (1, 1024, 1920, 40, 1e-10),   # 64 x 64 tiles, the inverse on their four wavefronts
    (1, 1024, 4096, 72, 1e-10),   # 64 x 128 tiles
])
def test_cache_factors_block_edges(B, M, d, r, ridge):
    """Edges of the 16-wide pivot blocks of the inverse and of the shares T comes in, against the
    oracle's fp64 solution for the G that the GPU stored."""
    Cm = wl.round_to_bf16(wl.cached_feature(B, M, d, r + 40, seed=290 + M, noise=0.1))
    Q = _q(B, M, r, 291 + M, "bf16", False)
    ctx = _ctx(d, "bf16")
    w_c = torch.full((B, M, r), float("nan"), dtype=torch.bfloat16, device="cuda")
    g_c = torch.full((B, r, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((fv.fvar_factors_workspace_bytes(ctx, B, M, r),), 0xff, dtype=torch.uint8, device="cuda")
    fv.fvar_cache_factors(ctx, to_dev(Cm, "bf16"), _qt_dev(Q, "bf16"), False, B, M, r, ridge, w_c, g_c, ws)
    torch.cuda.synchronize()
    Wg, Gg = to_np(w_c).astype(np.float64), to_np(g_c).astype(np.float64)
    for b in range(B):
        Wo = factors.restoration_matrix(Gg[b], Cm[b], ridge)     # against the G the GPU stored
        assert rel_err(Wg[b], Wo) <= TOL["bf16"], (b, rel_err(Wg[b], Wo))
        assert rel_err(Gg[b], factors.project(Q[0], Cm[b])) <= TOL["bf16"]


def _gram_matrices(kind, B, r, rng):
    """B badly conditioned matrices and their ridge, see test_gram_inverse_keeps_ill_conditioned_digits."""
    if kind == "diagonal":
        return np.stack([np.diag(10.0 ** rng.uniform(-6, 6, r)) for _ in range(B)]), 0.0
    if kind == "rank8+ridge":
        G, ridge = rng.standard_normal((B, r, min(r, 8))) @ rng.standard_normal((B, min(r, 8), 1024)), 1e-6
    else:
        G, ridge = np.abs(rng.standard_normal((B, r, 400))) @ np.abs(rng.standard_normal((B, 400, 2048))), 0.0
    return G @ G.transpose(0, 2, 1), ridge


def _check_inverse(kind, got, A0, ridge, rng):
    """One inverse against numpy's of A0 (the sum of the partial matrices) + ridge, with the bounds of
    test_gram_inverse_keeps_ill_conditioned_digits."""
    r = A0.shape[0]
    A = A0 + np.eye(r) * (ridge * np.trace(A0) / r)
    ref, cond = np.linalg.inv(A), np.linalg.cond(A)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    bound = 1e-15 if kind == "diagonal" else r * 2.0 ** -52 * cond
    assert err <= bound, f"cond {cond:.1e}: {err:.1e} > {bound:.1e}"
    if kind != "diagonal":
        Z = rng.standard_normal((40, r))
        W = Z - Z @ (A - A0) @ ref
        werr = np.linalg.norm(Z @ A0 @ got - W) / np.linalg.norm(W)
        assert werr <= bound, f"cond {cond:.1e}: T X off by {werr:.1e} > {bound:.1e}"


# (samples, rows, width, rank) -> rows per tile of T and its shares: every tile height with every instance of the
# inverse that its launch can hold
T_INVERSE = [((1, 256, 512, 8), 64, 1), ((1, 256, 512, 16), 128, 1), ((64, 1024, 2048, 16), 256, 1),
             ((1, 264, 4096, 32), 64, 3), ((3, 2304, 4096, 24), 128, 4),
             ((1, 256, 1920, 40), 64, 1), ((3, 256, 512, 56), 256, 1), ((1, 256, 512, 40), 128, 1), ((1, 512, 4096, 64), 128, 2),
             ((1, 256, 4096, 72), 64, 1), ((2, 256, 1920, 72), 128, 1), ((1, 256, 512, 104), 256, 1), ((4, 512, 4096, 128), 128, 1)]


@pytest.mark.parametrize("kind", ["rank8+ridge", "positive", "diagonal"])
@pytest.mark.parametrize("shape,tile,shares", T_INVERSE)
def test_inverse_inside_the_launch_of_t(shape, tile, shares, kind):
    """The bf16 path inverts inside T's launch, in the tiles' LDS and on as many wavefronts as they have: the same
    matrices and bounds as for the inverse by itself, in four partial sums, and T = C G^T beside it."""
    import ctypes as C
    B, M, d, r = shape
    rng = np.random.default_rng(M + r)
    lib = fv.load_library()
    assert lib["_ZN4fvar21batched_f32_tile_rowsEiiii"](B, M, r, d) == tile
    assert lib["_ZN4fvar17batched_f32_partsEiiii"](B, M, r, d) == shares
    n = min(B, 3)                                     # different matrices; sample b gets number b % n
    S, ridge = _gram_matrices(kind, n, r, rng)
    parts = np.stack([0.125 * S, 0.25 * S, 0.125 * S, 0.5 * S], axis=1)
    Sd = torch.from_numpy(np.ascontiguousarray(parts)).cuda()[torch.arange(B) % n].contiguous()
    g = torch.Generator(device="cuda").manual_seed(r)
    cache = torch.randn((B, M, d), generator=g, device="cuda").to(torch.bfloat16)
    G = torch.randn((B, r, d), generator=g, device="cuda").to(torch.bfloat16)
    T = torch.full((shares, B, M, r), float("nan"), device="cuda")
    X = torch.full((B, r, r), float("nan"), dtype=torch.float64, device="cuda")
    launch = lib["_ZN4fvar23launch_factor_t_inverseEPKvS1_iiiiPfPKddPdP12ihipStream_t"]
    launch.restype = None
    launch.argtypes = [C.c_void_p, C.c_void_p] + 4 * [C.c_int] + [C.c_void_p, C.c_void_p, C.c_double, C.c_void_p, C.c_void_p]
    torch.cuda.synchronize()
    launch(cache.data_ptr(), G.data_ptr(), B, M, r, d, T.data_ptr(), Sd.data_ptr(), ridge, X.data_ptr(), None)
    torch.cuda.synchronize()
    for b in sorted({0, 1, 2, B - 1} & set(range(B))):
        _check_inverse(kind, X[b].cpu().numpy(), parts[b % n].sum(0), ridge, rng)
        ref = cache[b].double() @ G[b].double().t()
        assert float((T[:, b].double().sum(0) - ref).norm() / ref.norm()) <= 1e-6    # fp32 sums of bf16 products


@pytest.mark.parametrize("r", [8, 16, 24, 32, 56, 64, 72, 104, 128])
@pytest.mark.parametrize("kind", ["rank8+ridge", "positive", "diagonal"])
def test_gram_inverse_keeps_ill_conditioned_digits(r, kind):
    """The inverse kernel by itself on badly conditioned matrices, in two partial sums.  Elimination in
    fp64 without pivoting is backward stable here, X = (S + E)^-1 with |E| <= r eps |S|, which bounds the
    inverse, |X - S^-1| <= r eps cond |S^-1|, and, far below |T| |X - S^-1|, the product T X with a T whose
    rows lie in the range of the large eigenvalues, as those of C G^T do: |T X - T S^-1| <= r eps cond
    |T S^-1|.  A block step by an explicit inverse breaks the first, an elimination whose triangles drift
    apart the second.  'diagonal' has a scaled identity: exact up to the division."""
    import ctypes as C
    rng = np.random.default_rng(r)
    B, ridge = 2, 0.0
    if kind == "rank8+ridge":
        G, ridge = rng.standard_normal((B, r, min(r, 8))) @ rng.standard_normal((B, min(r, 8), 1024)), 1e-6
    elif kind == "positive":
        G = np.abs(rng.standard_normal((B, r, 400))) @ np.abs(rng.standard_normal((B, 400, 2048)))
    S = np.stack([np.diag(10.0 ** rng.uniform(-6, 6, r)) for _ in range(B)]) if kind == "diagonal" else G @ G.transpose(0, 2, 1)
    parts = np.stack([0.25 * S, 0.75 * S], axis=1)
    Sd = torch.from_numpy(np.ascontiguousarray(parts)).cuda()
    X = torch.full((B, r, r), float("nan"), dtype=torch.float64, device="cuda")
    launch = fv.load_library()["_ZN4fvar21launch_factor_inverseEPKdiiidPdP12ihipStream_t"]
    launch.restype, launch.argtypes = None, [C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_double, C.c_void_p, C.c_void_p]
    torch.cuda.synchronize()
    launch(Sd.data_ptr(), 2, B, r, ridge, X.data_ptr(), None)
    torch.cuda.synchronize()
    for b in range(B):
        A = parts[b].sum(0)
        A = A + np.eye(r) * (ridge * np.trace(A) / r)
        ref, cond = np.linalg.inv(A), np.linalg.cond(A)
        got = X[b].cpu().numpy()
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        bound = 1e-15 if kind == "diagonal" else r * 2.0 ** -52 * cond
        assert err <= bound, (b, f"cond {cond:.1e}: {err:.1e} > {bound:.1e}")
        if kind != "diagonal":
            # T = Z S has T A^-1 = Z - Z (A - S) A^-1, without cancellation
            Z, S0 = rng.standard_normal((40, r)), parts[b].sum(0)
            W = Z - Z @ (A - S0) @ ref
            werr = np.linalg.norm(Z @ S0 @ got - W) / np.linalg.norm(W)
            assert werr <= bound, (b, f"cond {cond:.1e}: T X off by {werr:.1e} > {bound:.1e}")


@pytest.mark.parametrize("B,M,d,r", [(1, 1024, 1024, 64), (4, 4096, 4096, 128), (8, 4096, 4096, 128),
                                     (16, 4096, 4096, 64), (2, 1000, 1920, 24), (1, 72, 320, 8), (3, 520, 512, 128)])
def test_factor_t_rounding(B, M, d, r):
    """T = C G_c^T, which lies in the workspace as shares to be added up, against 64 bits, on positive values (every
    rounding counts).  A chain of n MFMAs is rounded at partial sums that have grown to i/n of its result, an
    rms of at most sqrt(n/3) 2^-24 of it; the d/(32 n) chains of a row are independent and their sum is
    compensated, so it and each addition of a share are one rounding more, at most 2^-24/sqrt(3) each.
    n is 8, or 4 where a share has no more than 16 k-tiles.  One chain per share
    breaks the bound at all of these, six-fold at d = 4096."""
    import ctypes as C
    rng = np.random.default_rng(M + r)
    cache = torch.from_numpy(np.abs(rng.standard_normal((M, 32)) @ rng.standard_normal((32, d))).astype(np.float32))
    cache = (cache * (1 + 0.1 * torch.arange(B)[:, None, None])).to(torch.bfloat16).cuda()
    qt = torch.from_numpy(np.abs(rng.standard_normal((r, M))).astype(np.float32) / r ** 0.5).to(torch.bfloat16).cuda()
    ctx = _ctx(d, "bf16")
    w_c = torch.empty((B, M, r), dtype=torch.bfloat16, device="cuda")
    g_c = torch.empty((B, r, d), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((fv.fvar_factors_workspace_bytes(ctx, B, M, r),), 0xff, dtype=torch.uint8, device="cuda")
    fv.fvar_cache_factors(ctx, cache, qt, False, B, M, r, 1e-6, w_c, g_c, ws)
    parts = fv.load_library()["_ZN4fvar14factor_t_partsENS_5DTypeEiiii"](C.c_int(1), B, M, r, d)
    shares = ws[:parts * B * M * r * 4].view(torch.float32).view(parts, B, M, r)
    T = shares[0].clone()
    for p in range(1, parts):
        T += shares[p]
    n = 8 if d / 64 / parts > 16 else 4
    bound = 2.0 ** -24 / 3 ** 0.5 * (n / max(1.0, d / (32 * n)) + parts) ** 0.5
    for b in range(B):
        ref = cache[b].double() @ g_c[b].double().t()
        err = ((T[b].double() - ref).norm() / ref.norm()).item()
        assert err <= bound, (b, parts, err, bound)


@pytest.mark.parametrize("dtype,steps", [("f32", ["project", "t", "gram", "inverse", "w"]),
                                         ("bf16", ["project", "gram", "t_inverse", "w"])])
def test_cache_factors_profile_names_every_step(dtype, steps):
    """Per-kernel timing of the factors: a label for each launch (bf16: T and the inverse share one)."""
    B, M, d, r = 1, 64, 64, 16
    ctx = _ctx(d, dtype)
    Cm, Q = wl.cached_feature(B, M, d, 20, seed=5, noise=0.1), _q(B, M, r, 6, dtype, False)
    w_c, g_c = (torch.empty(s, dtype=tdtype(dtype), device="cuda") for s in ((B, M, r), (B, r, d)))
    ws = torch.empty(fv.fvar_factors_workspace_bytes(ctx, B, M, r), dtype=torch.uint8, device="cuda")
    fv.fvar_profile_enable(ctx, True)
    fv.fvar_cache_factors(ctx, to_dev(Cm, dtype), _qt_dev(Q, dtype), False, B, M, r, 1e-6, w_c, g_c, ws)
    torch.cuda.synchronize()
    prof = fv.fvar_profile_read(ctx)
    assert sorted(prof) == sorted("factor_" + s for s in steps) and all(n == 1 and ms > 0 for n, ms in prof.values())


def test_cache_factors_feed_the_fill():
    # factors built on the GPU, used by the rank-r fill, against the oracle's fill of its factors
    dtype, B, M, d, r, k = "bf16", 2, 144, 256, 32, 58
    Cm = wl.round_to_bf16(wl.cached_feature(B, M, d, 40, seed=95, noise=0.05))
    Q = _q(B, M, r, 96, dtype, False)
    ctx = _ctx(d, dtype)
    w_c = torch.empty((B, M, r), dtype=torch.bfloat16, device="cuda")
    g_c = torch.empty((B, r, d), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(fv.fvar_factors_workspace_bytes(ctx, B, M, r), dtype=torch.uint8, device="cuda")
    fv.fvar_cache_factors(ctx, to_dev(Cm, dtype), _qt_dev(Q, dtype), False, B, M, r, 0.0, w_c, g_c, ws)
    rng = np.random.default_rng(1)
    keep = np.stack([np.sort(rng.choice(M, k, replace=False)) for _ in range(B)]).astype(np.int32)
    drop = np.stack([np.setdiff1d(np.arange(M), keep[b]) for b in range(B)]).astype(np.int32)
    yk = wl.activations_iid(B, k, d, seed=97, bf16=True)
    y = torch.empty((B, M, d), dtype=torch.bfloat16, device="cuda")
    fv.fvar_lowrank_fill(ctx, to_dev(yk, dtype), torch.from_numpy(keep).cuda(), torch.from_numpy(drop).cuda(),
                         B, M, k, r, w_c, g_c, y)
    torch.cuda.synchronize()
    for b in range(B):
        Wo, Go = factors.stored_factors(Cm[b], Q[0], bf16=True)
        ref = oracle.lowrank_fill(yk[b], keep[b], drop[b], M, Wo, Go)
        assert rel_err(to_np(y[b]), ref) <= TOL[dtype]


# ----------------------------------------------------------------------------- whole RP step
def _rp_case(dtype, B, M, r, d, H, Lp, seed):
    bf = dtype == "bf16"
    x = wl.activations_lowrank(B, M, d, seed=seed, bf16=bf)
    w = wl.block_weights(d, 4 * d, seed=seed + 1, bf16=bf, std=0.8 / np.sqrt(d))
    Kp, Vp = wl.kv_prefix(B, Lp, H, d // H, seed=seed + 2, bf16=bf)
    Cm = wl.cached_feature(B, M, d, max(8, r), seed=seed + 3, noise=0.05)
    if bf:
        Cm = wl.round_to_bf16(Cm)
    Q = _q(B, M, r, seed + 4, dtype, False)
    return x, w, Kp, Vp, Cm, Q


@pytest.mark.parametrize("dtype,B,M,r,d,H,Lp", [
    ("bf16", 2, 144, 58, 256, 4, 100),
    ("bf16", 1, 200, 64, 256, 2, 77),        # head_dim 128
    ("f32", 1, 64, 16, 128, 2, 40),
    ("f32", 1, 256, 128, 1024, 16, 424),     # the fp32 configuration with the projected input
])
def test_rp_step_parity(dtype, B, M, r, d, H, Lp):
    x, w, Kp, Vp, Cm, Q = _rp_case(dtype, B, M, r, d, H, Lp, seed=300 + M)
    blk = GpuBlock(d, H, 4 * d, dtype, w, Kp, Vp, Lp + r)
    xd = to_dev(x, dtype)
    f_r = torch.empty((B, r, d), dtype=tdtype(dtype), device="cuda")
    fv.fvar_rp_project(blk.ctx, _qt_dev(Q, dtype), False, xd, B, M, r, f_r)
    y_keep = blk.dense(f_r)                                  # the r projected rows are the block's tokens
    s, keep, drop = blk.score_select(xd, r)
    y = torch.full((B, M, d), float("nan"), dtype=tdtype(dtype), device="cuda")
    fv.fvar_cache_fill(blk.ctx, y_keep, keep, drop, B, M, r, to_dev(Cm, dtype), y)
    torch.cuda.synchronize()
    ow = oracle.BlockWeights(**w)
    for b in range(B):
        Kc = np.zeros((Lp + r, H, d // H), np.float32); Vc = np.zeros_like(Kc)
        Kc[:Lp], Vc[:Lp] = Kp[b], Vp[b]
        ref = rp_path.rp_step(x[b], Q[0], Cm[b], ow, H, Kc, Vc, Lp, bf16=dtype == "bf16")
        assert rel_err(to_np(f_r[b]), ref["f_r"]) <= TOL[dtype]
        assert np.array_equal(keep[b].cpu().numpy(), ref["idx_keep"])
        assert np.array_equal(drop[b].cpu().numpy(), ref["idx_drop"])
        assert rel_err(to_np(y_keep[b]), ref["y_keep"]) <= TOL[dtype], rel_err(to_np(y_keep[b]), ref["y_keep"])
        assert rel_err(to_np(blk.K[b, Lp:]), Kc[Lp:]) <= TOL[dtype]
        assert rel_err(to_np(blk.V[b, Lp:]), Vc[Lp:]) <= TOL[dtype]
        yg = to_np(y[b])
        assert np.array_equal(yg[ref["idx_drop"]], Cm[b][ref["idx_drop"]])
        assert np.array_equal(yg[ref["idx_keep"]], to_np(y_keep[b]))


def test_rp_project_depth30_launch_shape_sampled():
    # the shape the benchmark times (batch 8, scale 32, 410 of 1024 rows): sampled output rows
    W = wl.WORKLOADS["var_d30_512_bf16"]
    B, M, d = W.batch, W.tokens(32), W.hidden
    r = W.keep(32)
    x = wl.activations_lowrank(B, M, d, seed=1002, bf16=True)
    Q = _q(B, M, r, 4002, "bf16", False)
    ctx = _ctx(d, "bf16", H=W.heads)
    out = torch.empty((B, r, d), dtype=torch.bfloat16, device="cuda")
    fv.fvar_rp_project(ctx, _qt_dev(Q, "bf16"), False, to_dev(x, "bf16"), B, M, r, out)
    torch.cuda.synchronize()
    rng = np.random.default_rng(0)
    for b in (0, 3, 7):
        rows = np.concatenate([[0, r - 1, 127, 128, 383, 384], rng.integers(0, r, 10)])
        ref = Q[0][:, rows].astype(np.float64).T @ x[b].astype(np.float64)
        assert rel_err(to_np(out[b])[rows], factors.round_bf16(ref)) <= TOL["bf16"]


# ----------------------------------------------------------------------------- cache up-sampling
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,hs,ws,hd,wd,c", [(2, 3, 3, 4, 4, 8), (1, 24, 24, 32, 32, 64), (2, 5, 7, 8, 9, 24),
                                              (1, 4, 4, 4, 4, 16), (1, 6, 6, 3, 3, 8), (1, 1, 1, 5, 5, 8),
                                              (1, 18, 18, 24, 24, 1920)])
def test_upsample_tokens_parity(dtype, B, hs, ws, hd, wd, c):
    from oracle import upsample
    bf = dtype == "bf16"
    src = wl.activations_iid(B, hs * ws, c, seed=110 + hs, bf16=bf)
    ctx = _ctx(64, dtype)
    dst = torch.full((B, hd * wd, c), float("nan"), dtype=tdtype(dtype), device="cuda")
    fv.fvar_upsample_tokens(ctx, to_dev(src, dtype), B, hs, ws, c, hd, wd, dst)
    torch.cuda.synchronize()
    for b in range(B):
        ref = upsample.upsample_tokens(src[b], hs, ws, hd, wd)
        assert rel_err(to_np(dst[b]), ref) <= (2.0 ** -8 if bf else 1e-6)
    if (hs, ws) == (hd, wd):
        assert np.array_equal(to_np(dst), src)


@pytest.mark.parametrize("hs,hd,d,r,nblk,B,k", [(8, 12, 256, 32, 1, 2, 58),
                                               (24, 32, 1920, 64, 3, 2, 410),     # depth-30 shape, 24 -> 32
                                               (40, 48, 2048, 64, 2, 2, 692)])    # Infinity-2B shape, 40 -> 48
def test_factored_cache_handed_from_scale_to_scale(hs, hd, d, r, nblk, B, k):
    """The cached counterpart features stay in factored form between two scales: the outputs of
    all blocks at the previous scale are factored in ONE call (batch = blocks x samples), only the
    thin factor W_c is up-sampled to the next grid (Up(W_c G_c) = Up(W_c) G_c), and the next
    scale's restoration multiplies it with the unchanged G_c.  Against the oracle's chain
    stored_factors -> upsample_tokens -> lowrank_fill: every stage meets the bar on identical
    inputs (the oracle continues from the factors the GPU stored); the whole chain, in which the
    two sides may round a stored factor element to different bf16 neighbours before the rank-r sum
    amplifies the difference, is held to 2.5 x the bar, like the unrounded statement below."""
    from oracle import upsample
    dtype = "bf16"
    Ms, M, n = hs * hs, hd * hd, nblk * B
    Cm = wl.round_to_bf16(wl.cached_feature(n, Ms, d, max(r, 40), seed=120 + hs, noise=0.05))
    Q = _q(1, Ms, r, 121 + hs, dtype, False)
    ctx = _ctx(d, dtype)
    w_s = torch.empty((n, Ms, r), dtype=torch.bfloat16, device="cuda")
    g_c = torch.empty((n, r, d), dtype=torch.bfloat16, device="cuda")
    ws_ = torch.empty(fv.fvar_factors_workspace_bytes(ctx, n, Ms, r), dtype=torch.uint8, device="cuda")
    fv.fvar_cache_factors(ctx, to_dev(Cm, dtype), _qt_dev(Q, dtype), False, n, Ms, r, 0.0, w_s, g_c, ws_)
    w_up = torch.empty((n, M, r), dtype=torch.bfloat16, device="cuda")
    fv.fvar_upsample_tokens(ctx, w_s, n, hs, hs, r, hd, hd, w_up)
    rng = np.random.default_rng(2)
    keep = np.stack([np.sort(rng.choice(M, k, replace=False)) for _ in range(B)]).astype(np.int32)
    drop = np.stack([np.setdiff1d(np.arange(M), keep[b]) for b in range(B)]).astype(np.int32)
    yk = wl.activations_iid(B, k, d, seed=122, bf16=True)
    ykd, kd, dd = to_dev(yk, dtype), torch.from_numpy(keep).cuda(), torch.from_numpy(drop).cuda()
    torch.cuda.synchronize()
    Wg, Gg, Wupg = to_np(w_s), to_np(g_c), to_np(w_up)
    for i in range(n):                            # stage 1 and 2 against the oracle
        Wo, Go = factors.stored_factors(Cm[i], Q[0], bf16=True)
        assert rel_err(Gg[i], Go) <= TOL[dtype] and rel_err(Wg[i], Wo) <= TOL[dtype]
        assert rel_err(Wupg[i], upsample.upsample_tokens(Wg[i], hs, hs, hd, hd)) <= 2.0 ** -8
    for blk in range(nblk):                       # block blk of the next scale uses slice blk*B .. of the factors
        sl = slice(blk * B, (blk + 1) * B)
        y = torch.empty((B, M, d), dtype=torch.bfloat16, device="cuda")
        fv.fvar_lowrank_fill(ctx, ykd, kd, dd, B, M, k, r, w_up[sl].contiguous(), g_c[sl].contiguous(), y)
        torch.cuda.synchronize()
        for b in range(B):
            Wo, Go = factors.stored_factors(Cm[blk * B + b], Q[0], bf16=True)
            Wup = factors.round_bf16(upsample.upsample_tokens(Wo, hs, hs, hd, hd))
            ref = oracle.lowrank_fill(yk[b], keep[b], drop[b], M, Wup, Go)
            assert rel_err(to_np(y[b]), ref) <= 2.5 * TOL[dtype]                     # whole chain
            ref_stage = oracle.lowrank_fill(yk[b], keep[b], drop[b], M, Wupg[blk * B + b], Gg[blk * B + b])
            assert rel_err(to_np(y[b]), ref_stage) <= TOL[dtype]                    # stage 3 alone
            if blk == 0 and b == 0:
                # that restoration is the up-sampled restored cache itself; against this unrounded
                # statement the bf16 storage of Up(W_c) and of the output both count, hence the
                # wider bound
                full = upsample.upsample_tokens(Wo.astype(np.float64) @ Go.astype(np.float64), hs, hs, hd, hd)
                assert rel_err(to_np(y[b])[drop[b]], full[drop[b]]) <= 2.5 * TOL[dtype]


# ----------------------------------------------------------------------------- one selection per chunk
@pytest.mark.parametrize("dtype,B,M,k,d,H,Lp,r,nblk", [
    ("bf16", 2, 144, 58, 256, 4, 100, 16, 3),
    ("f32", 1, 64, 20, 128, 2, 40, 8, 2),
])
def test_block_chunk_with_one_selection(dtype, B, M, k, d, H, Lp, r, nblk):
    """Select once, gather once, run the chunk's blocks on the compact rows, fill once: the
    existing entry points chained (pruned call for the first block, the dense call on k rows for
    the others) against the oracle's chunk."""
    bf = dtype == "bf16"
    x = wl.activations_lowrank(B, M, d, seed=400, bf16=bf)
    ws = [wl.block_weights(d, 4 * d, seed=401 + i, bf16=bf, std=0.8 / np.sqrt(d)) for i in range(nblk)]
    kvs = [wl.kv_prefix(B, Lp, H, d // H, seed=420 + i, bf16=bf) for i in range(nblk)]
    Cm = wl.cached_feature(B, M, d, r, seed=430, noise=0.05)
    z = wl.normal_draws(B, M, r, seed=431)
    Wc = np.empty((B, M, r), np.float32); Gc = np.empty((B, r, d), np.float32)
    for b in range(B):
        Wc[b], Gc[b] = factors.cache_factors(Cm[b], z[b])
    if bf:
        Wc, Gc = wl.round_to_bf16(Wc), wl.round_to_bf16(Gc)
    blks = [GpuBlock(d, H, 4 * d, dtype, ws[i], kvs[i][0], kvs[i][1], Lp + k) for i in range(nblk)]
    xd = to_dev(x, dtype)
    s, keep, drop = blks[0].score_select(xd, k)
    rows = blks[0].pruned(xd, keep, k)
    for blk in blks[1:]:
        rows = blk.dense(rows)
    y = blks[0].fill(rows, keep, drop, M, to_dev(Wc, dtype), to_dev(Gc, dtype))
    torch.cuda.synchronize()
    for b in range(B):
        caches = []
        for i in range(nblk):
            Kc = np.zeros((Lp + k, H, d // H), np.float32); Vc = np.zeros_like(Kc)
            Kc[:Lp], Vc[:Lp] = kvs[i][0][b], kvs[i][1][b]
            caches.append((Kc, Vc))
        ref = oracle.pruned_chunk(x[b], k, [oracle.BlockWeights(**w) for w in ws], H, caches, Lp,
                                  Wc[b], Gc[b])
        assert np.array_equal(keep[b].cpu().numpy(), ref["idx_keep"])
        assert np.array_equal(drop[b].cpu().numpy(), ref["idx_drop"])
        assert rel_err(to_np(rows[b]), ref["y_keep"]) <= TOL[dtype], rel_err(to_np(rows[b]), ref["y_keep"])
        assert rel_err(to_np(y[b]), ref["y"]) <= TOL[dtype]
        for i in range(nblk):
            assert rel_err(to_np(blks[i].K[b, Lp:]), caches[i][0][Lp:]) <= TOL[dtype]
            assert rel_err(to_np(blks[i].V[b, Lp:]), caches[i][1][Lp:]) <= TOL[dtype]


def test_cache_factors_depth30_launch_shape():
    # the shape the benchmark times (batch 8, scale 32, rank 64): two samples against the oracle
    W = wl.WORKLOADS["var_d30_512_bf16"]
    B, M, d, r = W.batch, W.tokens(32), W.hidden, W.rank
    Cm = wl.round_to_bf16(wl.cached_feature(B, M, d, 180, seed=4100, noise=0.1))
    Q = _q(B, M, r, 4101, "bf16", False)
    ctx = _ctx(d, "bf16", H=W.heads)
    w_c = torch.empty((B, M, r), dtype=torch.bfloat16, device="cuda")
    g_c = torch.empty((B, r, d), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(fv.fvar_factors_workspace_bytes(ctx, B, M, r), dtype=torch.uint8, device="cuda")
    fv.fvar_cache_factors(ctx, to_dev(Cm, "bf16"), _qt_dev(Q, "bf16"), False, B, M, r, 0.0, w_c, g_c, ws)
    torch.cuda.synchronize()
    for b in (0, 7):
        Wo, Go = factors.stored_factors(Cm[b], Q[0], bf16=True)
        assert rel_err(to_np(g_c[b]), Go) <= TOL["bf16"]
        assert rel_err(to_np(w_c[b]), Wo) <= TOL["bf16"]


@pytest.mark.parametrize("B,M,d,r", [(200, 256, 512, 64), (192, 304, 448, 72), (96, 512, 1024, 128)])
def test_cache_factors_many_samples(B, M, d, r):
    """The caches of all blocks of a scale in one call (hundreds of samples): the projection
    G_c = Q^T C and the product T = C G_c^T then run on the tiled MFMA kernel of the linear
    layers (k-major operand / batched fp32 output).  Three samples against the oracle."""
    Cm = wl.round_to_bf16(wl.cached_feature(B, M, d, max(8, r // 2), seed=4300 + r, noise=0.1))
    Q = _q(B, M, r, 4301 + r, "bf16", False)
    ctx = _ctx(d, "bf16")
    w_c = torch.full((B, M, r), float("nan"), dtype=torch.bfloat16, device="cuda")
    g_c = torch.full((B, r, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(fv.fvar_factors_workspace_bytes(ctx, B, M, r), dtype=torch.uint8, device="cuda")
    fv.fvar_cache_factors(ctx, to_dev(Cm, "bf16"), _qt_dev(Q, "bf16"), False, B, M, r, 0.0, w_c, g_c, ws)
    torch.cuda.synchronize()
    assert torch.isfinite(w_c.float()).all() and torch.isfinite(g_c.float()).all()
    for b in (0, B // 3, B - 1):
        Wo, Go = factors.stored_factors(Cm[b], Q[0], bf16=True)
        assert rel_err(to_np(g_c[b]), Go) <= TOL["bf16"], (b, rel_err(to_np(g_c[b]), Go))
        assert rel_err(to_np(w_c[b]), Wo) <= TOL["bf16"], (b, rel_err(to_np(w_c[b]), Wo))


@pytest.mark.parametrize("r", [4, 12, 20, 36, 60, 68, 92, 100, 124])
@pytest.mark.parametrize("kind", ["rank8+ridge", "positive"])
def test_gram_inverse_at_ranks_of_four(r, kind):
    """Ranks that fp32 storage allows: the last group of four pivots ends a quarter, half or three quarters into its
    block of sixteen, in an odd or even number of tiles."""
    test_gram_inverse_keeps_ill_conditioned_digits(r, kind)
