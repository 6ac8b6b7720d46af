"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments before anything is launched."""
import ctypes as C
import os
import re

import pytest

import paper_2512_16483_amd as fv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "fvar.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fvar_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = fv.load_library()
    names = _declared()
    assert len(names) >= 13
    for n in names:
        assert hasattr(lib, n), f"{n} declared in fvar.h but not exported"
    assert sorted(fv.EXPORTS) == names


def test_keep_count_and_schedule_helpers():
    assert fv.fvar_keep_count(1600, 3, 10) == 480
    assert fv.fvar_keep_count(2304, 3, 10) == 692
    assert fv.fvar_keep_count(576, 2, 5) == 231
    assert fv.fvar_keep_count(10, 0, 7) == 1 and fv.fvar_keep_count(10, 9, 7) == 10
    assert fv.fvar_keep_count(0, 1, 2) == -1 and fv.fvar_keep_count(5, 1, 0) == -1
    c = fv.Context(hidden=2048, heads=16, head_dim=128, ffn_hidden=8192,
                   scales=(1, 2, 4, 6, 8, 12, 16, 20, 24, 32, 40, 48, 64))
    assert fv.fvar_scale_tokens(c, 12) == 4096 and fv.fvar_scale_prev_len(c, 12) == 6425
    assert fv.fvar_scale_prev_len(c, 10) == 2521 and fv.fvar_scale_tokens(c, 13) == -1
    r = fv.Context(hidden=128, heads=2, head_dim=64, ffn_hidden=256, scales=((3, 5), (4, 7)))
    assert fv.fvar_scale_tokens(r, 1) == 28 and fv.fvar_scale_prev_len(r, 1) == 15
    # workspace: four [rows,d] buffers, the fp32 residual stream [rows,d], one [rows,F] buffer and,
    # for a problem this small, 8 key-range partials of the attention ([rows,d] + 2 [rows,H] fp32)
    assert fv.fvar_block_workspace_bytes(r, 2, 10) == 4 * 5120 + 10240 + 10240 + 8 * 20 * (128 + 4) * 4
    big = fv.Context(hidden=1920, heads=30, head_dim=64, ffn_hidden=7680)
    rows = 8 * 410
    assert fv.fvar_block_workspace_bytes(big, 8, 410) == sum(
        (n + 255) // 256 * 256 for n in [rows * 1920 * 2] * 4 + [rows * 1920 * 4, rows * 7680 * 2])
    assert fv.fvar_select_workspace_bytes(r, 3, 100) == 1280


@pytest.mark.parametrize("kw", [
    dict(hidden=128, heads=3, head_dim=64, ffn_hidden=256),      # heads * head_dim != hidden
    dict(hidden=96, heads=3, head_dim=32, ffn_hidden=256),       # head_dim not 64 / 128
    dict(hidden=128, heads=2, head_dim=64, ffn_hidden=100),      # ffn not a multiple of 64
    dict(hidden=16384, heads=128, head_dim=128, ffn_hidden=256),  # row does not fit one wavefront
    dict(hidden=0, heads=0, head_dim=64, ffn_hidden=64),
])
def test_create_rejects_bad_geometry(kw):
    with pytest.raises(fv.FvarError):
        fv.Context(**kw)


def _call(lib, name, *args):
    return getattr(lib, name)(*args)


def test_entry_points_reject_bad_arguments_without_launching():
    lib = fv.load_library()
    c = fv.Context(hidden=128, heads=2, head_dim=64, ffn_hidden=256, dtype="bf16")
    h = c.handle
    fake = 0x1000          # aligned, never dereferenced on the host
    # k out of range, null outputs, misaligned pointer, missing workspace
    assert lib.fvar_score_select(h, None, fake, 1, 10, 11, None, None, fake, None, None, 0) == fv.FVAR_ERR_INVALID_ARG
    assert b"k<=M" in lib.fvar_last_error(h)
    assert lib.fvar_score_select(h, None, fake, 1, 10, 0, None, None, fake, None, None, 0) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_score_select(h, None, fake, 1, 10, 5, None, None, None, None, None, 0) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_score_select(h, None, None, 1, 10, 5, None, None, fake, None, None, 0) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_score_select(h, None, fake + 2, 1, 10, 5, None, None, fake, None, None, 0) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_score_select(h, None, fake, 1, 10, 5, None, None, fake, None, None, 0) == fv.FVAR_ERR_WORKSPACE
    assert lib.fvar_score_select(h, None, fake, 1, (1 << 20) + 1, 5, None, None, fake, None, fake, 1 << 30) == fv.FVAR_ERR_UNSUPPORTED

    w = fv._Weights()
    for n, _ in fv._Weights._fields_:
        setattr(w, n, None)
    kv = fv._KV(fake, fake, 100, 95)
    # weights missing
    assert lib.fvar_block_forward_pruned(h, None, C.byref(w), fake, 1, 10, fake, 5, C.byref(kv), fake, fake, 1 << 30) == fv.FVAR_ERR_INVALID_ARG
    for n in ("w_qkv", "w_o", "w_fc1", "w_fc2"):
        setattr(w, n, fake)
    # cache overflow: len 95 + 10 rows > capacity 100
    assert lib.fvar_block_forward_dense(h, None, C.byref(w), fake, 1, 10, C.byref(kv), fake, fake, 1 << 30) == fv.FVAR_ERR_INVALID_ARG
    assert b"capacity" in lib.fvar_last_error(h)
    kv.len = 0
    # k > M, NULL index list with k < M, workspace too small
    assert lib.fvar_block_forward_pruned(h, None, C.byref(w), fake, 1, 10, fake, 11, C.byref(kv), fake, fake, 1 << 30) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_block_forward_pruned(h, None, C.byref(w), fake, 1, 10, None, 5, C.byref(kv), fake, fake, 1 << 30) == fv.FVAR_ERR_INVALID_ARG
    need = fv.fvar_block_workspace_bytes(c, 1, 5)
    assert lib.fvar_block_forward_pruned(h, None, C.byref(w), fake, 1, 10, fake, 5, C.byref(kv), fake, fake, need - 1) == fv.FVAR_ERR_WORKSPACE
    assert lib.fvar_block_forward_pruned(h, None, C.byref(w), fake, 1, 10, fake, 5, C.byref(kv), fake, None, 0) == fv.FVAR_ERR_WORKSPACE
    # fill: rank must be a multiple of 8 for bf16 and at most 256; factors required when k < M
    assert lib.fvar_lowrank_fill(h, None, fake, fake, fake, 1, 10, 5, 12, fake, fake, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_lowrank_fill(h, None, fake, fake, fake, 1, 10, 5, 264, fake, fake, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_lowrank_fill(h, None, fake, fake, fake, 1, 10, 5, 16, None, fake, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_lowrank_fill(h, None, fake, fake, None, 1, 10, 5, 16, fake, fake, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_lowrank_fill(h, None, fake, fake, fake, 1, 10, 11, 16, fake, fake, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_status_string(fv.FVAR_ERR_WORKSPACE) == b"workspace too small"
    # random projection: rows in [1,M], M a multiple of 8 for bf16, pointers present and aligned
    assert lib.fvar_rp_project(h, None, fake, 0, fake, 1, 16, 17, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_rp_project(h, None, fake, 0, fake, 1, 16, 0, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_rp_project(h, None, None, 0, fake, 1, 16, 4, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_rp_project(h, None, fake + 4, 0, fake, 1, 16, 4, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_rp_project(h, None, fake, 0, fake, 1, 12, 4, fake) == fv.FVAR_ERR_UNSUPPORTED
    # raw-cache fill: the cache and the pruned index list are required when rows are pruned
    assert lib.fvar_cache_fill(h, None, fake, fake, fake, 1, 10, 11, fake, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_cache_fill(h, None, fake, fake, None, 1, 10, 5, fake, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_cache_fill(h, None, fake, fake, fake, 1, 10, 5, None, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_cache_fill(h, None, None, fake, fake, 1, 10, 5, fake, fake) == fv.FVAR_ERR_INVALID_ARG
    # up-sampling: sizes >= 1, channels a multiple of the 16-byte chunk
    assert lib.fvar_upsample_tokens(h, None, fake, 1, 0, 4, 8, 8, 8, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_upsample_tokens(h, None, None, 1, 4, 4, 8, 8, 8, fake) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_upsample_tokens(h, None, fake, 1, 4, 4, 12, 8, 8, fake) == fv.FVAR_ERR_UNSUPPORTED
    # factors: rank limits, ridge sign, workspace
    need = fv.fvar_factors_workspace_bytes(c, 2, 64, 16)
    assert need == 2 * 2 * 64 * 16 * 4 + (8 + 1) * (2 * 16 * 16 * 8)     # 2 slices of T, 8 partial Gram matrices, inverse
    assert lib.fvar_cache_factors(h, None, fake, fake, 0, 2, 64, 136, 0.0, fake, fake, fake, 1 << 30) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_cache_factors(h, None, fake, fake, 0, 2, 256, 136, 0.0, fake, fake, fake, 1 << 30) == fv.FVAR_ERR_UNSUPPORTED
    assert lib.fvar_cache_factors(h, None, fake, fake, 0, 2, 64, 12, 0.0, fake, fake, fake, 1 << 30) == fv.FVAR_ERR_UNSUPPORTED
    assert lib.fvar_cache_factors(h, None, fake, fake, 0, 2, 64, 16, -1.0, fake, fake, fake, 1 << 30) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_cache_factors(h, None, fake, fake, 0, 2, 64, 16, 0.0, fake, None, fake, 1 << 30) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_cache_factors(h, None, fake, fake, 0, 2, 64, 16, 0.0, fake, fake, fake, need - 1) == fv.FVAR_ERR_WORKSPACE


def test_block_calls_reject_operands_beyond_32bit_tile_offsets():
    """The linear-layer kernels address an operand matrix with 32-bit byte offsets: a call whose
    widest operand (B*rows x max(hidden, ffn_hidden) elements) reaches 4 GiB must be refused
    before anything is launched, not wrap silently."""
    lib = fv.load_library()
    c = fv.Context(hidden=2048, heads=16, head_dim=128, ffn_hidden=8192, dtype="bf16")
    h, fake = c.handle, 0x1000
    w = fv._Weights()
    for n, _ in fv._Weights._fields_:
        setattr(w, n, None)
    for n in ("w_qkv", "w_o", "w_fc1", "w_fc2"):
        setattr(w, n, fake)
    kv = fv._KV(fake, fake, 1 << 20, 0)
    # 64 x 4096 rows x 8192 columns x 2 bytes = 4 GiB exactly: refused
    assert lib.fvar_block_forward_dense(h, None, C.byref(w), fake, 64, 4096, C.byref(kv), fake, fake, 1 << 60) == fv.FVAR_ERR_UNSUPPORTED
    assert b"4 GiB" in lib.fvar_last_error(h)
    # one row less per sample is inside the limit: the call gets as far as the workspace check
    assert lib.fvar_block_forward_dense(h, None, C.byref(w), fake, 64, 4095, C.byref(kv), fake, fake, 16) == fv.FVAR_ERR_WORKSPACE
    # batch beyond the launch grid's third dimension (8 key ranges per sample)
    assert lib.fvar_block_forward_dense(h, None, C.byref(w), fake, 8192, 8, C.byref(kv), fake, fake, 1 << 60) == fv.FVAR_ERR_UNSUPPORTED
    # the selection without workspace: size limit and argument checks need no GPU either
    assert lib.fvar_score_select_static(h, None, fake, 1025, 1024, 4, fake, None) == fv.FVAR_ERR_UNSUPPORTED
    assert lib.fvar_score_select_static(h, None, fake, 1, 8, 9, fake, None) == fv.FVAR_ERR_INVALID_ARG
    assert lib.fvar_debug_checks(h, 1) == fv.FVAR_OK and lib.fvar_debug_checks(h, 0) == fv.FVAR_OK


def test_missing_library_fails_loudly(monkeypatch):
    monkeypatch.setattr(fv, "_lib", None)
    monkeypatch.setattr(fv, "LIB_PATH", "/nonexistent/libfvar.so")
    with pytest.raises(ImportError):
        fv.load_library()


class _Plan(C.Structure):
    _fields_ = [("cfg", C.c_int), ("nsplit", C.c_int), ("tail", C.c_int), ("scratch_floats", C.c_size_t)]


class _BlockPlan(C.Structure):
    _fields_ = [("layer", _Plan * 4), ("floats", C.c_size_t)]


def block_plan(dtype, B, n, d, H, F):
    """How a block's linear layers run (an internal function of the library; pure host code)."""
    f = fv.load_library()["_ZN4fvar10block_planENS_5DTypeEiiiiii"]
    f.restype, f.argtypes = _BlockPlan, [C.c_int] * 7
    return f(1 if dtype == "bf16" else 0, B, n, d, H, d // H, F)


TILES = ("320x256", "256x256", "192x256", "256x192", "256x128", "128x256", "192x128", "128x128", "64x128", "128x64", "64x64")
RINGS = ("16x16", "32x16", "16x32", "32x32", "48x32", "32x64", "64x64", "48x64")     # features x rows of a workgroup
LAYERS = ("qkv", "o", "fc1", "fc2")


def linear_plans(dtype, B, n, d, H, F):
    """{layer: (tile or ring instance, shares, last round's shares)} of a block as it runs."""
    return {l: (TILES[p.cfg] if p.cfg < len(TILES) else "ring " + RINGS[p.cfg - len(TILES)], p.nsplit, p.tail)
            for l, p in zip(LAYERS, block_plan(dtype, B, n, d, H, F).layer)}


@pytest.mark.parametrize("B,n,d,H,F,layer,tile,shares,last_round", [
    (1, 64, 2048, 16, 8192, "qkv", "ring 48x32", 1, 1),
    (1, 64, 2048, 16, 8192, "fc2", "ring 32x64", 4, 1),
    (2, 65, 1024, 16, 4096, "fc1", "ring 64x64", 1, 1),
    (1, 257, 1024, 16, 4096, "fc1", "128x64", 1, 1),
    (1, 257, 1024, 16, 4096, "fc2", "64x128", 6, 1),
    (1, 257, 128, 2, 256, "fc2", "64x64", 1, 1),
    (1, 700, 1024, 16, 4096, "fc1", "128x128", 1, 1),
    (1, 700, 1024, 16, 4096, "fc2", "128x128", 5, 1),
    (4, 225, 1920, 30, 7680, "qkv", "192x128", 1, 1),
    (4, 225, 1920, 30, 7680, "fc1", "128x256", 1, 1),
    (2, 924, 1920, 15, 7680, "qkv", "256x192", 1, 1),
    (2, 924, 1920, 15, 7680, "fc1", "256x256", 1, 1),
    (3, 25, 3072, 48, 64, "qkv", "128x128", 3, 1),
    (4, 36, 4096, 32, 1024, "qkv", "192x128", 2, 1),
    (3, 214, 4096, 32, 64, "qkv", "128x256", 1, 8),
    (3, 214, 4096, 32, 64, "fc1", "64x64", 8, 1),
    (2, 805, 4096, 32, 64, "qkv", "256x256", 1, 3),
    (1, 180, 1536, 24, 5440, "fc2", "64x128", 7, 1),
])
def test_plans_that_the_gpu_tests_are_there_for(B, n, d, H, F, layer, tile, shares, last_round):
    """tests/test_gpu_linear_plans.py runs the block at these row counts: another choice of constants must not
    take a kernel, a tile or a division out of its reach unseen."""
    assert linear_plans("bf16", B, n, d, H, F)[layer] == (tile, shares, last_round)


@pytest.mark.parametrize("rows,d,layer,tile,shares", [
    (703, 1536, "fc2", "192x128", 5), (776, 1280, "fc2", "192x128", 5), (1229, 1024, "fc2", "128x128", 3),
    (300, 4096, "o", "192x128", 4), (421, 3072, "o", "128x64", 1),       # 64x64: more workgroups than CUs, hence no groups
])
def test_plan_prices_the_kernel_that_is_launched(rows, d, layer, tile, shares):
    """Tiles with wavefront groups have time constants of their own, which hold only where the launch uses groups.
    These picks measured 22 to 31 % less time than those of a plan that prices both kernels alike."""
    assert linear_plans("bf16", 1, rows, d, d // 64, 4 * d)[layer] == (tile, shares, 1)


# Microseconds of a layer of few rows, weights from HBM: by the plan that had no kernel with rings per wavefront (fp32: by
# the kernel that loaded its operands straight to registers), and by candidates of now.
FEW_ROWS = [
    ("bf16", 7, 4096, 16384, "fc2", 33.2, {("ring 16x16", 1): 39.4, ("ring 32x16", 2): 27.2, ("ring 32x32", 2): 27.4}),
    ("bf16", 16, 4096, 16384, "fc2", 33.4, {("ring 16x16", 1): 40.0, ("ring 32x16", 2): 27.6, ("ring 32x32", 2): 27.4}),
    ("bf16", 24, 4096, 16384, "fc2", 34.4, {("ring 32x32", 1): 47.0, ("ring 32x32", 2): 28.5}),
    ("bf16", 32, 4096, 16384, "fc2", 34.4, {("ring 32x32", 1): 49.0, ("ring 32x32", 2): 29.3, ("ring 64x64", 4): 30.5}),
    ("bf16", 32, 4096, 16384, "fc1", 31.5, {("ring 32x32", 1): 33.2, ("ring 64x64", 1): 27.6}),
    ("bf16", 32, 3072, 16384, "fc2", 27.7, {("ring 32x16", 1): 35.0, ("ring 48x32", 4): 24.1}),
    ("bf16", 24, 3072, 16384, "fc2", 27.5, {("ring 32x16", 1): 33.2, ("ring 48x32", 4): 23.6}),
    ("bf16", 12, 3072, 12288, "fc1", 21.3, {("64x64", 1): 21.5, ("ring 48x32", 1): 15.2}),
    ("bf16", 48, 1920, 7680, "fc2", 14.1, {("ring 64x64", 8): 14.8, ("ring 32x64", 4): 13.5}),
    ("bf16", 4, 2048, 8192, "fc1", 9.1, {("ring 16x16", 1): 9.9, ("ring 32x16", 1): 8.2, ("ring 32x32", 1): 8.3}),
    ("f32", 4, 1024, 8192, "fc1", 10.2, {("ring 16x16", 1): 11.5, ("ring 32x16", 1): 9.8}),
    ("f32", 16, 1024, 8192, "fc1", 10.7, {("ring 16x16", 1): 11.5, ("ring 32x16", 1): 9.5}),
]


@pytest.mark.parametrize("dtype,rows,d,F,layer,before,now", FEW_ROWS)
def test_few_rows_take_no_slower_kernel(dtype, rows, d, F, layer, before, now):
    """The kernel with a ring per wavefront is for the rows where it is the faster one."""
    pick = linear_plans(dtype, 1, rows, d, d // (64 if d < 2048 else 128), F)[layer]
    assert now[pick[:2]] <= before, pick


@pytest.mark.parametrize("B,rows,d,H,most", [(4, 38, 1024, 16, 6225920), (8, 19, 1024, 16, 6225920), (3, 51, 1024, 16, 6364928),
                                             (16, 47, 512, 8, 12320768), (2, 64, 1536, 24, 8650752),
                                             (16, 37, 832, 13, 13791232), (8, 52, 1600, 25, 23961600)])
def test_bf16_block_workspace_stays_within_what_callers_were_told(B, rows, d, H, most):
    """Programs that keep the size of an earlier library must not be refused."""
    c = fv.Context(hidden=d, heads=H, head_dim=64, ffn_hidden=4 * d, dtype="bf16")
    assert fv.fvar_block_workspace_bytes(c, B, rows) <= most


def test_shares_and_tiles_of_the_factor_tests():
    """tests/test_gpu_rp_path.py covers T = C G^T in one to four shares, on 64, 128 and 256 rows per tile, with each
    instance of the inverse: another choice of constants must not empty these cases unseen."""
    lib = fv.load_library()
    tile, parts = lib["_ZN4fvar21batched_f32_tile_rowsEiiii"], lib["_ZN4fvar17batched_f32_partsEiiii"]
    for (B, M, d, r), expect in {(1, 1024, 4096, 64): (128, 2), (1, 264, 4096, 32): (64, 3), (1, 520, 4096, 8): (64, 4),
                                 (1, 1024, 1920, 40): (64, 1), (1, 1024, 4096, 72): (64, 1), (1, 4096, 4096, 128): (128, 1),
                                 (2, 1000, 1920, 24): (64, 2)}.items():
        assert (tile(B, M, r, d), parts(B, M, r, d)) == expect, (B, M, d, r)


def test_projection_groups_only_where_tiles_share_what_they_read():
    """Wavefront groups in the small projection tile gain where few column strips are read at once; many samples,
    or a few k-tiles, are faster without (512 samples of 256 x 1024: 80 us instead of 90)."""
    groups = fv.load_library()["_ZN4fvar16kmajor_in_groupsEiiii"]
    groups.restype = C.c_bool
    for B, M, rows, d, expect in ((1, 2304, 692, 2048, True), (1, 2312, 692, 2048, True), (16, 4096, 64, 1024, True),
                                  (8, 2304, 120, 2048, True), (1, 512, 40, 1024, True), (1, 448, 40, 1024, False),
                                  (24, 1024, 64, 1024, False), (512, 256, 16, 1024, False), (64, 4096, 64, 1024, False),
                                  (1, 128, 40, 2048, False), (1, 4096, 2000, 2048, False)):
        assert groups(B, M, rows, d) == expect, (B, M, rows, d)


def test_fill_runs_in_one_round_of_workgroups():
    """Two workgroups of the fill fit a CU at every rank: more than 512 of them are a second round, unless the slabs
    alone are more.  Every 32-row group has a workgroup's wavefront, and no workgroup goes without."""
    split = fv.load_library()["_ZN4fvar14fill_row_splitEii"]
    for slabs in list(range(1, 70)) + [105, 120, 224, 256, 257, 511, 512, 513, 1024]:      # all samples' together
        for nd in (0, 1, 32, 33, 128, 129, 700, 1120, 4800):
            n = split(slabs, nd)
            assert (nd == 0 and n == 0) or 1 <= n <= max(1, 512 // slabs)
            assert (n - 1) * 128 < max(nd, 1) and (n == 512 // slabs or n * 128 >= nd or n == 1)


def test_fill_keeps_maps_in_cache_that_the_next_block_reads_there():
    """A restored map is read again by the next block's score pass: it goes past the caches only where it is small
    or does not fit the 256 MB of last-level cache."""
    past = fv.load_library()["_ZN4fvar15map_past_cachesEmb"]
    past.restype, past.argtypes = C.c_bool, [C.c_size_t, C.c_bool]
    for mb, plain, scored in ((1, True, True), (19, True, True), (31, False, True), (52, False, False),
                              (105, False, False), (210, False, False), (302, False, False), (420, True, True), (5000, True, True)):
        assert (past(mb * 10 ** 6, False), past(mb * 10 ** 6, True)) == (plain, scored), mb


@pytest.mark.parametrize("B,n,d,H,F,layer,tile,shares", [
    (3, 90, 1088, 17, 1088, "qkv", "64x64", 1), (1, 520, 960, 15, 2240, "fc2", "64x64", 1),
    (1, 257, 512, 8, 1088, "fc2", "64x64", 1),
    (1, 330, 1088, 17, 4096, "fc1", "128x64", 1), (1, 400, 960, 15, 4160, "fc2", "128x64", 4),
    (3, 100, 2048, 16, 2112, "qkv", "64x128", 1),
])
def test_plans_of_the_wavefront_group_tests(B, n, d, H, F, layer, tile, shares):
    """tests/test_gpu_linear_plans.py runs these blocks for the tiles whose k-tiles are dealt to groups."""
    N, K = {"qkv": (3 * d, d), "fc1": (F, d), "fc2": (d, F)}[layer]
    assert linear_plans("bf16", B, n, d, H, F)[layer] == (tile, shares, 1)
    bm, bn = map(int, tile.split("x"))
    workgroups, per = -(-B * n // bm) * -(-N // bn) * shares, -(-K // 64 // shares)
    assert per >= (32 if tile == "64x128" else 16) and (tile != "64x64" or workgroups <= 256)


@pytest.mark.parametrize("d,H,F", [(1024, 16, 4096), (512, 8, 5440), (64, 1, 64), (4096, 32, 4096)])
def test_f32_block_workspace_grows_with_the_call(d, H, F):
    """fp32 callers may size one workspace for their largest scale: the size never falls as the rows or
    the batch grow."""
    c = fv.Context(hidden=d, heads=H, head_dim=d // H, ffn_hidden=F, dtype="f32")
    for B in (1, 2, 3, 8):
        last = 0
        for n in list(range(1, 700)) + list(range(700, 5000, 37)):
            need = fv.fvar_block_workspace_bytes(c, B, n)
            assert last <= need <= fv.fvar_block_workspace_bytes(c, B + 1, n), (B, n, last, need)
            last = need


@pytest.mark.parametrize("dtype,d,H", [("f32", 1024, 16), ("bf16", 1024, 16), ("bf16", 1920, 30), ("bf16", 4096, 32)])
def test_block_workspace_holds_the_partial_results(dtype, d, H):
    """What the workspace has besides the activations is enough for the plan of every linear layer and
    for the attention, which use it in turn."""
    F, es, al = 4 * d, 2 if dtype == "bf16" else 4, lambda n: -(-n // 256) * 256
    c = fv.Context(hidden=d, heads=H, head_dim=d // H, ffn_hidden=F, dtype=dtype)
    att = fv.load_library()["_ZN4fvar24attention_scratch_floatsENS_5DTypeEiiii"]
    att.restype = C.c_size_t
    for B in (1, 3, 32):
        for n in list(range(1, 260, 3)) + [363, 640, 1021, 1537, 1600, 2048, 3122]:
            R = B * n
            part = fv.fvar_block_workspace_bytes(c, B, n) - 4 * al(R * d * es) - al(R * d * 4) - al(R * F * es)
            plans = block_plan(dtype, B, n, d, H, F).layer
            held = [p.nsplit * R * N if p.nsplit > 1 else 0 for p, N in zip(plans, (3 * d, d, F, d))]
            held += [p.scratch_floats for p in plans] + [att(1 if dtype == "bf16" else 0, B, n, H, d // H)]
            assert part >= 4 * max(held), (B, n)


@pytest.mark.parametrize("dtype,d", [("f32", 512), ("bf16", 128), ("bf16", 1024), ("bf16", 1920), ("bf16", 4096)])
def test_factors_workspace_grows_with_the_call(dtype, d):
    """The workspace of fvar_cache_factors never shrinks as rows, samples or rank grow, and holds every share
    that T comes in."""
    c = fv.Context(hidden=d, heads=d // 64, head_dim=64, ffn_hidden=d, dtype=dtype)
    parts = fv.load_library()["_ZN4fvar14factor_t_partsENS_5DTypeEiiii"]
    size = fv.fvar_factors_workspace_bytes
    for B in (1, 2, 4, 8, 16, 40):
        for r in (8, 64, 128):
            last, gram = 0, 9 * (-(-8 * B * r * r // 256) * 256) if dtype == "bf16" else 2 * (-(-8 * B * r * r // 256) * 256)
            for M in list(range(128, 4300, 56)) + [4096, 4104] + list(range(4304, 30000, 808)):
                if M == 4096:
                    last = 0
                need = size(c, B, M, r)
                assert last <= need <= min(size(c, B + 1, M, r), size(c, B, M, r + 8)), (B, M, r, last, need)
                assert need - gram >= 4 * parts(C.c_int(1 if dtype == "bf16" else 0), B, M, r, d) * B * M * r
                last = need


@pytest.mark.parametrize("dtype,B,n,d,H,F,expect", [
    ("f32", 3, 6, 1024, 8, 4096, [("16x32", 1), ("16x16", 1), ("16x32", 1), ("16x32", 4)]),
    ("f32", 5, 50, 320, 5, 1280, [("32x32", 1), ("16x32", 1), ("32x64", 1), ("16x32", 1)]),
    ("f32", 1, 85, 960, 15, 3840, [("48x32", 1), None, None, ("48x32", 4)]),
    ("f32", 1, 200, 1024, 16, 4096, [("48x64", 1), ("32x32", 1), ("64x64", 1), None]),
    ("f32", 1, 3, 2048, 32, 64, [None, None, ("16x16", 8), None]),
    ("f32", 1, 33, 768, 12, 5440, [None, None, None, ("48x32", 8)]),
    ("f32", 1, 57, 1088, 17, 5440, [None, None, None, ("32x32", 2)]),
    ("bf16", 1, 43, 1536, 24, 6144, [("48x32", 1), None, None, ("48x32", 4)]),
    ("bf16", 1, 99, 1536, 24, 6144, [("48x64", 1), None, None, ("48x64", 4)]),
    ("bf16", 1, 141, 4096, 32, 1024, [None, None, ("32x32", 1), ("64x64", 1)]),
    ("bf16", 7, 14, 1024, 16, 4096, [("48x32", 1), ("16x32", 1), ("32x64", 1), None]),
    ("bf16", 1, 48, 1920, 30, 7680, [("48x32", 1), ("16x32", 1), ("32x64", 1), ("32x64", 4)]),
    ("bf16", 1, 33, 1920, 30, 7680, [None, None, None, ("64x64", 8)]),
    ("bf16", 1, 3, 768, 12, 8192, [None, None, None, ("32x16", 8)]),
    ("bf16", 3, 8, 4096, 32, 16384, [None, None, ("64x64", 1), ("32x32", 2)]),
    ("bf16", 2, 65, 1024, 16, 4096, [("48x64", 1), ("32x32", 1), None, ("32x32", 1)]),
])
def test_instances_of_the_ring_kernel(dtype, B, n, d, H, F, expect):
    """tests/test_gpu_linear_plans.py is there for these."""
    got = linear_plans(dtype, B, n, d, H, F)
    assert all(e is None or got[l] == ("ring " + e[0], e[1], 1) for l, e in zip(LAYERS, expect)), got


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_plans_that_run_stay_within_the_workspace(dtype):
    """Every call gets a plan whose partial results fit what its workspace has besides the activations."""
    es, al = 2 if dtype == "bf16" else 4, lambda n: -(-n // 256) * 256
    for d, H, F in ((64, 1, 64), (192, 3, 256), (1024, 16, 4096), (1920, 30, 7680), (4096, 32, 1024), (4096, 32, 16384)):
        c = fv.Context(hidden=d, heads=H, head_dim=d // H, ffn_hidden=F, dtype=dtype)
        for B, n in ((1, 1), (1, 15), (3, 11), (1, 100), (2, 128), (1, 257), (4, 700), (32, 1600)):
            R = B * n
            part = fv.fvar_block_workspace_bytes(c, B, n) - 4 * al(R * d * es) - al(R * d * 4) - al(R * F * es)
            for p, N in zip(block_plan(dtype, B, n, d, H, F).layer, (3 * d, d, F, d)):
                assert p.scratch_floats >= (p.nsplit * R * N if p.nsplit > 1 else 0)
                assert 4 * p.scratch_floats <= part, (d, B, n, N)
                assert p.cfg < len(TILES) + len(RINGS) and (p.cfg >= len(TILES) or dtype == "bf16")


@pytest.mark.parametrize("B,n,d,H,F,expect", [
    (1, 436, 768, 12, 3072, ("64x64", 3)), (4, 100, 512, 8, 2048, ("64x64", 4)),
    (1, 72, 1920, 30, 7680, ("128x64", 8)), (1, 137, 1536, 24, 6144, ("64x128", 7)),
    (1, 180, 1536, 24, 5440, ("64x128", 7)),
])
def test_small_tiles_in_shares_stay_in_reach(B, n, d, H, F, expect):
    """tests/test_gpu_linear_plans.py runs these for the division of small tiles (their FC2)."""
    assert linear_plans("bf16", B, n, d, H, F)["fc2"] == expect + (1,)


@pytest.mark.parametrize("dtype,N,cfg,nsplit,tail", [
    ("bf16", 1024, len(TILES) + 7, 1, 1), ("bf16", 2048, len(TILES) + 4, 1, 1),      # 48 features do not divide N
    ("bf16", 1920, len(TILES) + len(RINGS), 1, 1), ("bf16", 1920, -1, 1, 1), ("f32", 1920, len(TILES) + len(RINGS), 1, 1),
    ("f32", 1024, len(TILES) + 7, 1, 1), ("f32", 1920, 4, 1, 1),                     # tiles are bf16 only
    ("bf16", 1920, 10, 0, 1), ("bf16", 1920, 10, 1, 0),
])
def test_plans_that_cannot_be_launched_are_refused(dtype, N, cfg, nsplit, tail):
    """Such a plan would leave columns unwritten: the launcher says so and launches nothing."""
    f = fv.load_library()["_ZN4fvar11launch_gemmENS_5DTypeEPKvS2_iiiRKNS_12GemmEpilogueERKNS_8GemmPlanEPfP12ihipStream_t"]
    f.restype = C.c_bool
    epilogue, plan = C.create_string_buffer(256), _Plan(cfg, nsplit, tail, 0)
    null = C.c_void_p(None)
    assert f(1 if dtype == "bf16" else 0, null, null, 64, N, 1920, epilogue, C.byref(plan), null, null) is False


@pytest.mark.parametrize("B,n,L,H,Dh,groups,ranges", [
    (2, 2, 635, 32, 128, 1, 2),       # 12.7 us; two groups without ranges 15.0
    (5, 18, 1271, 30, 64, 1, 3),      # 14.8; 17.2
    (1, 17, 582, 32, 128, 1, 2),      # 12.1; 13.7
    (3, 2, 944, 30, 64, 1, 3),        # 11.4; two groups, two ranges 12.7
    (3, 25, 567, 16, 128, 1, 2),      # 12.9; undivided 14.2
    (6, 3, 910, 16, 128, 1, 3),       # 16.6; two groups, two ranges 18.1
    (2, 142, 519, 30, 64, 1, 2),      # 15.6; undivided 16.5
    (2, 1024, 2521, 16, 128, 2, 1),   # 50.6; three ranges 65.4
    (8, 231, 871, 30, 64, 2, 1),
])
def test_attention_is_divided_as_measured(B, n, L, H, Dh, groups, ranges):
    """Few queries over a short cache: a division that is not the faster one (microseconds above) is not taken."""
    assert fv.load_library()["_ZN4fvar14attention_waysEiiiii"](B, n, L, H, Dh) == 100 * groups + ranges
