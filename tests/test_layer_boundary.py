"""Host-side checks of the layer entry points (include/ssa_layer.h): argument
validation happens before any HIP call, so it runs without a GPU; the split-K
workspace rule.  No GPU."""
import ctypes

import pytest

from paper_2606_05933_amd import ssa

LIB = ssa.LIB
NULL = ctypes.c_void_p(None)


def ws(m, n, k):
    out = ctypes.c_size_t(0)
    rc = LIB.ssa_linear_workspace_size(m, n, k, ctypes.byref(out))
    return rc, out.value


@pytest.mark.parametrize("m,n,k", [(-1, 128, 64), (4, 100, 64), (4, 128, 65), (4, 0, 64),
                                   (4, 128, 0), (2 ** 31 - 1, 1 << 20, 64)])
def test_linear_rejects_bad_sizes(m, n, k):
    assert ws(m, n, k)[0] == ssa.SSA_ERR_ARG
    assert LIB.ssa_linear(m, n, k, 0, NULL, NULL, NULL, NULL, NULL, 0, NULL) == ssa.SSA_ERR_ARG


def test_linear_rejects_a_bad_epilogue_and_null_pointers():
    assert LIB.ssa_linear(4, 128, 64, 3, NULL, NULL, NULL, NULL, NULL, 0, NULL) == ssa.SSA_ERR_ARG
    assert LIB.ssa_linear(4, 128, 64, 0, NULL, NULL, NULL, NULL, NULL, 0, NULL) == ssa.SSA_ERR_NULL
    # an empty product needs no pointers
    assert LIB.ssa_linear(0, 128, 64, 0, NULL, NULL, NULL, NULL, NULL, 0, NULL) == ssa.SSA_OK


def test_linear_workspace_rule():
    # enough 128 x 128 tiles to fill the chip: one pass over K, no workspace
    assert ws(2048, 4096, 4096) == (0, 0)
    assert ws(0, 4096, 4096) == (0, 0)
    # a decode-only batch: few tiles, K split; tickets (256 B) + fp32 partial
    # tiles, at most one per 256 of K for each of the M x N outputs' tiles
    rc, b = ws(28, 6144, 4096)
    assert rc == 0 and b > 256 and (b - 256) % (4 * 6144) == 0
    assert b - 256 <= 4 * 6144 * 256 * (4096 // 256)


@pytest.mark.parametrize("m,n,k", [(1, 1 << 30, 64), (31, 2 ** 31 - 128, 64), (32, 1 << 30, 64),
                                   (40, 1 << 30, 64), (64, 1 << 29, 256), (1, 2 ** 31 - 128, 512),
                                   (2 ** 24, 2048, 64), (2 ** 28, 128, 64), (1500, 1 << 25, 64)])
def test_linear_plans_the_largest_sizes_as_launches_the_runtime_takes(m, n, k):
    """A launch holds fewer than 2^32 threads; every size that is taken gets tiles
    whose grid does."""
    p = ssa.linear_plan(m, n, k)
    assert p.tiles_m == -(-m // p.tile_m) and p.tiles_n * p.tile_n == n
    assert p.tiles_m * p.tiles_n * p.splits * p.threads < 2 ** 32


def test_gpu_cases_cover_the_linear_tile_configurations():
    """Every tile configuration, with one and with several M tiles, unsplit and
    K-split, is in the sizes that test_gpu_gemm.py compares with the oracle: a change
    of the rule that picks them must not drop one."""
    from test_gpu_gemm import CASES, TILE_EDGES
    tiles = [(32, 64, 256), (64, 64, 256), (64, 128, 256), (96, 64, 256), (96, 128, 256),
             (128, 64, 256), (128, 128, 512), (160, 128, 256), (192, 128, 256), (192, 128, 512),
             (256, 128, 512), (256, 256, 512)]
    want = {t + (many, split) for t in tiles for many in (False, True) for split in (False, True)}
    have, split_tiles = set(), 0
    for m, n, k, _ in CASES + TILE_EDGES:
        p = ssa.linear_plan(m, n, k)
        have.add((p.tile_m, p.tile_n, p.threads, p.tiles_m > 1, p.splits > 1))
        if p.splits > 1:
            split_tiles = max(split_tiles, p.tiles_m * p.tiles_n)
    assert want <= have, sorted(want - have)
    assert split_tiles > 256  # the upper split tickets of a word


def test_linear_plan_checks_its_arguments():
    out = ssa.SsaLinearPlanInfo()
    assert LIB.ssa_linear_plan(4, 100, 64, ctypes.byref(out)) == ssa.SSA_ERR_ARG
    assert LIB.ssa_linear_plan(4, 128, 64, None) == ssa.SSA_ERR_NULL
    assert LIB.ssa_linear_plan(0, 128, 64, ctypes.byref(out)) == ssa.SSA_OK
    assert (out.tile_m, out.tiles_m, out.splits) == (0, 0, 0)


@pytest.mark.parametrize("m,n,k", [(28, 6144, 4096), (1, 128, 8192), (128, 4096, 14336)])
def test_linear_refuses_a_small_product_without_its_workspace(m, n, k):
    rc, need = ws(m, n, k)
    assert rc == 0 and need > 0
    fake = ctypes.c_void_p(1 << 40)
    for buf, nbytes in ((NULL, need), (fake, need - 1), (fake, 0)):
        assert LIB.ssa_linear(m, n, k, 0, fake, fake, NULL, fake, buf, ctypes.c_size_t(nbytes),
                              NULL) == ssa.SSA_ERR_WORKSPACE


def test_rms_norm_rejects_bad_arguments():
    f = ctypes.c_float
    assert LIB.ssa_rms_norm(4, 12, NULL, NULL, f(1e-5), NULL, NULL) == ssa.SSA_ERR_ARG
    assert LIB.ssa_rms_norm(4, 8200, NULL, NULL, f(1e-5), NULL, NULL) == ssa.SSA_ERR_ARG
    assert LIB.ssa_rms_norm(4, 64, NULL, NULL, f(-1.0), NULL, NULL) == ssa.SSA_ERR_ARG
    assert LIB.ssa_rms_norm(4, 64, NULL, NULL, f(float("nan")), NULL, NULL) == ssa.SSA_ERR_ARG
    assert LIB.ssa_rms_norm(4, 64, NULL, NULL, f(1e-5), NULL, NULL) == ssa.SSA_ERR_NULL
    assert LIB.ssa_rms_norm(0, 64, NULL, NULL, f(1e-5), NULL, NULL) == ssa.SSA_OK


def layer_args(hidden=256, inter=256, max_position=64, q_len=(5, 1), ctx_len=(10, 40)):
    """A host plan of a small batch and a weights struct of dummy device pointers
    (validation never dereferences them)."""
    import numpy as np
    shape = ssa.make_shape(4, 2, 64, 64, 8, 0.125)
    plan, _ = ssa.ssa_plan(shape, np.array(q_len, np.int32), np.array(ctx_len, np.int32))
    fake = ctypes.c_void_p(1 << 40)
    w = ssa.SsaLayerWeights(fake, fake, fake, fake, fake, fake, fake, hidden, inter,
                            max_position, 1e-5)
    return shape, plan, w, fake


def forward(shape, plan, w, fake, ws_bytes):
    return LIB.ssa_layer_forward(ctypes.byref(shape), ctypes.c_void_p(plan.ctypes.data), fake,
                                 ctypes.byref(w), fake, fake, fake, fake, fake, fake, ws_bytes,
                                 NULL)


def layer_ws(shape, plan, w):
    out = ctypes.c_size_t(0)
    rc = LIB.ssa_layer_workspace_size(ctypes.byref(shape), ctypes.c_void_p(plan.ctypes.data),
                                      ctypes.byref(w), ctypes.byref(out))
    return rc, out.value


def test_layer_workspace_holds_the_activations():
    shape, plan, w, _ = layer_args()
    rc, b = layer_ws(shape, plan, w)
    # 6 tokens: xn, h (hidden), qkv ((4 + 2 * 2) * 64), q and attention out (4 * 64), act
    assert rc == ssa.SSA_OK and b >= 6 * 2 * (256 * 2 + 512 + 256 * 2 + 256)


@pytest.mark.parametrize("hidden,inter", [(200, 256), (8320, 256), (256, 100), (256, 0)])
def test_layer_rejects_bad_sizes(hidden, inter):
    shape, plan, w, fake = layer_args(hidden=hidden, inter=inter)
    assert layer_ws(shape, plan, w)[0] == ssa.SSA_ERR_ARG
    assert forward(shape, plan, w, fake, 1 << 30) == ssa.SSA_ERR_ARG


def test_layer_rejects_positions_past_the_rotary_table_and_a_small_workspace():
    shape, plan, w, fake = layer_args(max_position=40)  # position 40 needs 41 rows
    assert forward(shape, plan, w, fake, 1 << 30) == ssa.SSA_ERR_ARG
    shape, plan, w, fake = layer_args(max_position=41)
    _, need = layer_ws(shape, plan, w)
    assert forward(shape, plan, w, fake, need - 1) == ssa.SSA_ERR_WORKSPACE


def test_layer_rejects_null_pointers_and_accepts_an_empty_batch():
    shape, plan, w, fake = layer_args()
    w.w_down = None
    assert forward(shape, plan, w, fake, 1 << 30) == ssa.SSA_ERR_NULL
    # no new tokens: nothing to launch, so no buffer is needed but the plan
    shape, plan, w, fake = layer_args(q_len=(0, 0))
    rc = LIB.ssa_layer_forward(ctypes.byref(shape), ctypes.c_void_p(plan.ctypes.data), fake,
                               ctypes.byref(w), NULL, NULL, NULL, NULL, NULL, NULL, 0, NULL)
    assert rc == ssa.SSA_OK
