"""fp32 FullyConnected in one launch with the whole reduction of a 16 x 16 tile in one workgroup (fc_few_f32) against the CPU
oracle, |gpu - oracle| <= 1e-5 + 1e-4 |oracle|: every number of wavefronts, ragged rows, columns and reductions, one trip and
several; which calls take it, with the same answer from the query as before."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl

SHAPES = [(1, 1, 1), (3, 5, 17), (16, 16, 16), (17, 47, 33), (2, 192, 40), (1, 2048, 1000), (33, 193, 16), (40, 769, 65), (5, 1027, 100),
          (129, 301, 77)]


@pytest.mark.parametrize("tile", range(3))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_fc_few(shape, tile, knobs):
    import gpu_util as G
    m, k, n = shape
    knobs.set("F32_FC_FEW", 2)
    knobs.set("F32_FC_FEW_TILE", tile)
    rng = np.random.default_rng(39000 + m + k + n)
    a = rng.uniform(-1, 1, size=(m, k)).astype(np.float32)
    w = (rng.uniform(-1, 1, size=(k, n)) / np.sqrt(k)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(n,)).astype(np.float32)
    for bias, act in ((b, wl.ACT_RELU), (None, wl.ACT_NONE)):
        got, variant = G.gpu_fc_f32(a, w, bias, act)
        assert variant.endswith("_w%d" % (4, 8, 16)[tile]), variant
        G.assert_close_f32(got, oracle.fc_f32(a, w, bias, act=act), f"{shape} [{variant}]")


@pytest.mark.parametrize("k", [30, 47, 64])
def test_non_finite_rows_stay_to_themselves(k, knobs):
    """A reduction that ends inside a lane's four indices: what lies behind it in the input is the next row."""
    import gpu_util as G
    knobs.set("F32_FC_FEW", 2)
    rng = np.random.default_rng(39100 + k)
    a, w = rng.uniform(-1, 1, size=(20, k)).astype(np.float32), rng.uniform(-1, 1, size=(k, 24)).astype(np.float32)
    a[5, 0], a[9, 1], a[17, 0] = np.inf, np.nan, -np.inf
    for tile in range(3):
        knobs.set("F32_FC_FEW_TILE", tile)
        got, _ = G.gpu_fc_f32(a, w, None, wl.ACT_NONE)
        rows = [r for r in range(20) if r not in (5, 9, 17)]
        G.assert_close_f32(got[rows], oracle.fc_f32(a[rows], w, None, act=wl.ACT_NONE), f"{k} {tile}")
        assert not np.isfinite(got[[5, 9, 17]]).any()


@pytest.mark.parametrize("shape,taken", [((2, 480, 208), True), ((1, 2048, 1000), True), ((21, 920, 2224), True), ((125, 784, 320), True),
                                         ((2, 2048, 1000), True), ((4, 1600, 744), True),
                                         ((4, 2048, 1000), True), ((1, 3072, 1000), True),      # on tiles of 8 x 8 and 4 x 4; 16 x 16 left them
                                         ((44, 456, 4280), False), ((16, 248, 64), False), ((16, 256, 64), True), ((40, 256, 64), True), ((256, 4096, 4096), False), ((9, 5088, 112), False)], ids=str)
def test_which_calls_take_it(shape, taken, knobs):
    import torch
    import gpu_util as G
    import paper_1805_00907_amd as glowmi
    m, k, n = shape
    a, w = torch.randn((m, k), device="cuda:0"), torch.randn((k, n), device="cuda:0")
    y = G.poison((m, n), torch.float32)
    need = glowmi.fc_workspace_bytes(m, k, n)
    variants = []
    for ws in (None, G.workspace(need)):
        glowmi.fc(a, w, None, y, m, k, n, wl.ACT_NONE, ws)
        variants.append(glowmi.last_variant())
    assert variants[1].startswith("fc_few_f32_w") == taken, variants
    assert not taken or variants[0] == variants[1]
    if taken:                                            # (all below the static buffer's limit)
        glowmi.fc_noalloc(a, w, None, y, m, k, n)
        assert glowmi.last_variant() == variants[1]
    torch.cuda.synchronize()
    knobs.set("F32_FC_FEW", 0)
    assert glowmi.fc_workspace_bytes(m, k, n) == need


@pytest.mark.parametrize("tile", range(3, 7))
@pytest.mark.parametrize("shape", SHAPES + [(9, 1025, 9), (4, 130, 4), (8, 2049, 71)], ids=lambda s: "x".join(map(str, s)))
def test_smaller_tiles(shape, tile, knobs):
    """Tiles of 8 x 8 and 4 x 4: sets of indices side by side in one matrix instruction; infinities and NaNs stay in their rows."""
    import gpu_util as G
    m, k, n = shape
    knobs.set("F32_FC_FEW", 2)
    knobs.set("F32_FC_FEW_TILE", tile)
    rng = np.random.default_rng(39200 + m + k + n)
    a = rng.uniform(-1, 1, size=(m, k)).astype(np.float32)
    w = (rng.uniform(-1, 1, size=(k, n)) / np.sqrt(k)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(n,)).astype(np.float32)
    for bias, act in ((b, wl.ACT_RELU), (None, wl.ACT_NONE)):
        got, variant = G.gpu_fc_f32(a, w, bias, act)
        assert variant == "fc_few_f32_" + ("w8c8", "w16c8", "w4c4", "w8c4")[tile - 3], variant
        G.assert_close_f32(got, oracle.fc_f32(a, w, bias, act=act), f"{shape} [{variant}]")
    if m > 2:
        a[1, 0], a[m - 1, k - 1] = np.nan, np.inf
        got, _ = G.gpu_fc_f32(a, w, b, wl.ACT_NONE)
        rows = [r for r in range(m) if r not in (1, m - 1)]
        G.assert_close_f32(got[rows], oracle.fc_f32(a[rows], w, b, act=wl.ACT_NONE), f"{shape} [{variant}] other rows")
        assert not np.isfinite(got[[1, m - 1]]).any()


@pytest.mark.parametrize("shape,variant", [((4, 2048, 1000), "fc_few_f32_w16c8"), ((1, 2048, 1000), "fc_few_f32_w8c4"), ((1, 1696, 544), "fc_few_f32_w8c4"),
                                           ((1, 512, 1000), "fc_rows_f32"), ((16, 4096, 4096), "fc_skinny16_f32")], ids=str)
def test_which_calls_take_smaller_tiles(shape, variant):
    """The answer of the query stays that of the kernel they stand in for."""
    import torch
    import gpu_util as G
    import paper_1805_00907_amd as glowmi
    m, k, n = shape
    rng = np.random.default_rng(39300 + m + k + n)
    a, w = rng.standard_normal((m, k), dtype=np.float32), (rng.standard_normal((k, n), dtype=np.float32) / np.sqrt(k)).astype(np.float32)
    got, took = G.gpu_fc_f32(a, w, None, wl.ACT_NONE)
    assert took.startswith(variant), took
    G.assert_close_f32(got, oracle.fc_f32(a, w, None, act=wl.ACT_NONE), took)
    need = glowmi.fc_workspace_bytes(m, k, n)
    glowmi.tuning_set("F32_FC_FEW", 0)
    try:
        assert glowmi.fc_workspace_bytes(m, k, n) == need
    finally:
        glowmi.tuning_reset()
