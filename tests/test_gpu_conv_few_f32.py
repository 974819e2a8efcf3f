"""The fp32 kernel for convolutions on few pixels with any reduction (conv_few_f32: four to sixteen wavefronts share the reduction
of a tile of 16 pixels x 16 or 32 channels, one launch, no workspace; in one form the tile's input patch lies in LDS) through the C ABI against the CPU oracle, element by element,
|gpu - oracle| <= 1e-5 + 1e-4 |oracle|: every tile form, ragged pixels, channels and reductions, one and several passes over
the reduction, taps on padding, with and without the add link, in place too."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


def _gpu():
    import gpu_util
    return gpu_util


# n  h  w  c  k  r  s  stride  pads(t,l,b,r)
SHAPES = [
    (1, 1, 1, 4, 1, 1, 1, (1, 1), (0, 0, 0, 0)),           # one output, a quarter of one group of indices
    (1, 5, 5, 12, 17, 3, 3, (1, 1), (1, 1, 1, 1)),         # groups of sixteen across taps, channels that end inside four
    (2, 4, 4, 16, 16, 1, 1, (1, 1), (0, 0, 0, 0)),         # whole tiles, one group: all wavefronts but one idle
    (2, 7, 9, 256, 40, 3, 3, (1, 1), (1, 1, 1, 1)),        # 2304 indices
    (1, 11, 6, 100, 33, 3, 3, (2, 1), (0, 1, 2, 1)),       # 900: the last group is not whole, one-sided padding
    (3, 3, 3, 36, 66, 5, 4, (2, 2), (2, 3, 2, 2)),         # most taps on padding
    (1, 6, 6, 1032, 24, 1, 1, (1, 1), (0, 0, 0, 0)),
    (1, 3, 5, 520, 20, 3, 3, (1, 1), (1, 1, 1, 1)),        # 4680: several passes in every form
    (1, 9, 13, 64, 31, 1, 1, (2, 2), (0, 0, 0, 0)),
    (2, 17, 5, 68, 47, 3, 3, (1, 2), (1, 1, 1, 1)),        # a chunk of four channels behind two whole ones, a wavefront with two chunks
    (1, 2, 33, 192, 18, 1, 3, (1, 1), (0, 1, 0, 1)),       # one row of taps
    (2, 5, 7, 3, 21, 3, 3, (1, 1), (1, 1, 1, 1)),          # channels that are no multiple of four: value by value
    (1, 6, 5, 43, 18, 1, 1, (1, 1), (0, 0, 0, 0)),
    (1, 4, 6, 131, 35, 3, 3, (2, 2), (1, 1, 1, 1)),        # 1179 indices, several passes
]


@pytest.mark.parametrize("tile", range(4))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:7])))
def test_conv_few(shape, tile, knobs):
    G = _gpu()
    n, h, w, c, k, r, s, st, pd = shape
    knobs.set("F32_FEW", 2)
    knobs.set("F32_FEW_TILE", tile)
    rng = np.random.default_rng(38000 + c + k)
    x = rng.uniform(-1, 1, size=(n, h, w, c)).astype(np.float32)
    wt = (rng.uniform(-1, 1, size=(k, r, s, c)) / np.sqrt(r * s * c)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(k,)).astype(np.float32)
    desc = G.make_desc(x.shape, wt.shape, st, pd, 1)
    for act, bias in ((wl.ACT_RELU, b), (wl.ACT_NONE, None)):
        ref = oracle.conv2d_f32(x, wt, bias, st, pd, 1, act=act)
        got, variant = G.gpu_conv2d_f32(x, wt, bias, desc, act)
        assert variant.startswith("conv_few_f32"), variant
        if tile == 3 and r * s > 1 and c % 4 == 0:             # the patch in LDS
            assert variant == "conv_few_f32_taps", variant
        G.assert_close_f32(got, ref, f"{shape} act {act} [{variant}]")
        add = rng.uniform(-1, 1, size=ref.shape).astype(np.float32)
        ref = oracle.conv2d_f32_add(x, wt, bias, add, st, pd, 1, act=act)
        for in_place in (False, True):
            got, variant = G.gpu_conv2d_f32_chain(x, wt, bias, add, desc, act, in_place=in_place)
            assert variant.startswith("conv_few_f32"), variant
            G.assert_close_f32(got, ref, f"{shape} add act {act} [{variant}]")


@pytest.mark.parametrize("c,r", [(13, 1), (13, 3), (20, 3)])
def test_conv_few_non_finite_filter_stays_in_its_channel(c, r, knobs):
    """A reduction that ends inside a lane's four indices: what lies behind it in the filter is the next channel."""
    G = _gpu()
    knobs.set("F32_FEW", 2)
    rng = np.random.default_rng(38900 + c)
    x = rng.uniform(-1, 1, size=(1, 5, 6, c)).astype(np.float32)
    wt = rng.uniform(-1, 1, size=(9, r, r, c)).astype(np.float32)
    wt[4, 0, 0, 0], wt[6, 0, 0, 1] = np.inf, np.nan
    desc = G.make_desc(x.shape, wt.shape, (1, 1), (r // 2,) * 4, 1)
    ref = oracle.conv2d_f32(x, wt, None, (1, 1), (r // 2,) * 4, 1, act=wl.ACT_NONE)
    for tile in range(3):
        knobs.set("F32_FEW_TILE", tile)
        got, variant = G.gpu_conv2d_f32(x, wt, None, desc, wl.ACT_NONE)
        assert variant.startswith("conv_few_f32"), variant
        keep = [k for k in range(9) if k not in (4, 6)]
        G.assert_close_f32(got[..., keep], np.ascontiguousarray(ref[..., keep]), f"{c} {r} [{variant}]")
        assert not np.isfinite(got[..., [4, 6]][~np.isfinite(ref[..., [4, 6]])]).any()


@pytest.mark.parametrize("few", [0, 1])
@pytest.mark.parametrize("shape", [(1, 56, 56, 256, 64, 1, 1), (1, 56, 56, 64, 64, 3, 1), (2, 9, 11, 16, 20, 3, 1), (1, 13, 7, 128, 36, 1, 1),
                                   (1, 12, 12, 64, 40, 3, 2), (4, 7, 7, 24, 68, 3, 1), (1, 1, 1, 128, 4, 1, 1)], ids=str)
def test_conv_small_both_forms(shape, few, knobs):
    """The layers of conv_small_f32 by its own kernel and by the one that the planner may take in its place."""
    G = _gpu()
    n, h, w, c, k, r, st = shape
    knobs.set("F32_FEW", few)
    rng = np.random.default_rng(38800 + c + k)
    x = rng.uniform(-1, 1, size=(n, h, w, c)).astype(np.float32)
    wt = (rng.uniform(-1, 1, size=(k, r, r, c)) / np.sqrt(r * r * c)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(k,)).astype(np.float32)
    pd = (r // 2,) * 4
    ref = oracle.conv2d_f32(x, wt, b, (st, st), pd, 1, act=wl.ACT_RELU)
    for ws in (True, False):
        got, variant = G.gpu_conv2d_f32(x, wt, b, G.make_desc(x.shape, wt.shape, (st, st), pd, 1), wl.ACT_RELU, use_workspace=ws)
        assert variant == "conv_small_f32" if not few else variant.startswith(("conv_small_f32", "conv_few_f32")), variant
        G.assert_close_f32(got, ref, f"{shape} few {few}")
