"""The fp32 kernel for pointwise convolutions on many pixels (conv_short_f32) through the C ABI against the CPU oracle: every slice
width, ragged pixels, channels and reductions, trips past the reduction, several blocks to a wavefront, strides, with and without
the add link, in place too; an infinity reaches the outputs of its own pixel and no other; and what the planner gives it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


def _gpu():
    import gpu_util
    return gpu_util


# n  h  w  c  k  stride
SHAPES = [
    (1, 1, 1, 4, 1, (1, 1)),             # one output, a quarter of a step
    (1, 5, 7, 20, 33, (1, 1)),           # a step of four channels, a tile of one channel
    (2, 4, 8, 64, 64, (1, 1)),           # whole blocks, tiles and trips
    (3, 9, 13, 72, 130, (1, 1)),         # a trip that is half past the reduction
    (1, 11, 6, 100, 37, (2, 1)),
    (2, 9, 14, 16, 200, (2, 3)),
    (1, 33, 31, 196, 96, (1, 1)),        # seven trips
]


@pytest.mark.parametrize("tiles", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:5])))
def test_conv_short_f32(shape, tiles, knobs):
    G = _gpu()
    n, h, w, c, k, st = shape
    knobs.set("F32_SHORT", 2)
    knobs.set("F32_SHORT_FORM", tiles)
    rng = np.random.default_rng(42000 + c + k)
    x = rng.uniform(-1, 1, size=(n, h, w, c)).astype(np.float32)
    wt = (rng.uniform(-1, 1, size=(k, 1, 1, c)) / np.sqrt(c)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(k,)).astype(np.float32)
    desc = G.make_desc(x.shape, wt.shape, st, (0, 0, 0, 0), 1)
    taken = "conv_short_f32" if 3 * tiles * 32 * ((c + 31) // 32 * 64 + 16) + tiles * 128 <= 160 * 1024 else ""
    for act, bias in ((wl.ACT_RELU, b), (wl.ACT_NONE, None)):
        ref = oracle.conv2d_f32(x, wt, bias, st, (0, 0, 0, 0), 1, act=act)
        for ws in (True, False):
            got, variant = G.gpu_conv2d_f32(x, wt, bias, desc, act, use_workspace=ws)
            assert variant.startswith(taken), variant
            G.assert_close_f32(got, ref, f"{shape} act {act} [{variant}]")
        add = rng.uniform(-1, 1, size=ref.shape).astype(np.float32)
        ref = oracle.conv2d_f32_add(x, wt, bias, add, st, (0, 0, 0, 0), 1, act=act)
        for in_place in (False, True):
            got, variant = G.gpu_conv2d_f32_chain(x, wt, bias, add, desc, act, in_place=in_place)
            assert variant.startswith(taken), variant
            G.assert_close_f32(got, ref, f"{shape} add act {act} [{variant}]")


@pytest.mark.parametrize("c,k,n,h,add,taken", [(64, 32, 2, 128, False, True), (128, 31, 1, 182, False, True), (64, 3, 1, 256, True, False), (128, 20, 1, 256, True, True),
                                               (64, 33, 2, 128, False, False), (64, 32, 1, 257, False, False), (128, 8, 2, 222, False, True)])
def test_narrow_layers_are_planned(c, k, n, h, add, taken):
    """Up to 32 channels over 64 or 128: at most 2048 blocks of 32 pixels or 3072 and more, fours with an addend."""
    G = _gpu()
    rng = np.random.default_rng(42700 + c + k + h)
    x = rng.uniform(-1, 1, size=(n, h, h, c)).astype(np.float32)
    wt = (rng.uniform(-1, 1, size=(k, 1, 1, c)) / np.sqrt(c)).astype(np.float32)
    desc = G.make_desc(x.shape, wt.shape, (1, 1), (0, 0, 0, 0), 1)
    if add:
        extra = rng.uniform(-1, 1, size=(n, h, h, k)).astype(np.float32)
        ref = oracle.conv2d_f32_add(x, wt, None, extra, (1, 1), (0, 0, 0, 0), 1, act=wl.ACT_RELU)
        got, variant = G.gpu_conv2d_f32_chain(x, wt, None, extra, desc, wl.ACT_RELU)
    else:
        ref = oracle.conv2d_f32(x, wt, None, (1, 1), (0, 0, 0, 0), 1, act=wl.ACT_RELU)
        got, variant = G.gpu_conv2d_f32(x, wt, None, desc, wl.ACT_RELU)
    assert variant.startswith("conv_short_f32" if taken else "conv_pw_f32"), variant
    G.assert_close_f32(got, ref, f"{c} {k} [{variant}]")


@pytest.mark.parametrize("c,k,h,add", [(24, 184, 60, False), (56, 224, 60, True), (224, 56, 75, False), (16, 40, 110, True)])
def test_conv_short_f32_is_planned(c, k, h, add):
    """Several blocks to a wavefront, with and without a workspace."""
    G = _gpu()
    rng = np.random.default_rng(42500 + c)
    x = rng.uniform(-1, 1, size=(3, h, h, c)).astype(np.float32)
    wt = (rng.uniform(-1, 1, size=(k, 1, 1, c)) / np.sqrt(c)).astype(np.float32)
    desc = G.make_desc(x.shape, wt.shape, (1, 1), (0, 0, 0, 0), 1)
    extra = rng.uniform(-1, 1, size=(3, h, h, k)).astype(np.float32)
    if add:
        ref = oracle.conv2d_f32_add(x, wt, None, extra, (1, 1), (0, 0, 0, 0), 1, act=wl.ACT_RELU)
        got, variant = G.gpu_conv2d_f32_chain(x, wt, None, extra, desc, wl.ACT_RELU)
    else:
        ref = oracle.conv2d_f32(x, wt, None, (1, 1), (0, 0, 0, 0), 1, act=wl.ACT_RELU)
        got, variant = G.gpu_conv2d_f32(x, wt, None, desc, wl.ACT_RELU)
    assert variant.startswith("conv_short_f32"), variant
    G.assert_close_f32(got, ref, f"{c} {k} [{variant}]")


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_conv_short_f32_non_finite(value, knobs):
    """One bad value at the end of a pixel's channels: its pixel's outputs are not finite, all others as without it."""
    G = _gpu()
    knobs.set("F32_SHORT", 2)
    rng = np.random.default_rng(42600)
    x = rng.uniform(-1, 1, size=(1, 7, 9, 20)).astype(np.float32)
    wt = rng.uniform(0.1, 1, size=(40, 1, 1, 20)).astype(np.float32)
    desc = G.make_desc(x.shape, wt.shape, (1, 1), (0, 0, 0, 0), 1)
    clean, _ = G.gpu_conv2d_f32(x, wt, None, desc, wl.ACT_NONE)
    x[0, 3, 4, 19] = value
    got, variant = G.gpu_conv2d_f32(x, wt, None, desc, wl.ACT_NONE)
    assert variant.startswith("conv_short_f32"), variant
    assert not np.isfinite(got[0, 3, 4]).any()
    got[0, 3, 4] = clean[0, 3, 4]
    assert np.array_equal(got, clean)


@pytest.mark.parametrize("tiles", [1, 2, 3, 4])
@pytest.mark.parametrize("add", [False, True])
def test_conv_short_f32_non_finite_results_are_those_of_fp32_arithmetic(tiles, add, knobs):
    """Infinities keep their sign, inf - inf and 0 * inf are NaN, values that bf16 would round to infinity stay finite; in the
    input, in the filter, at the ends of blocks and tiles, with the add link in place."""
    G = _gpu()
    knobs.set("F32_SHORT", 2)
    knobs.set("F32_SHORT_FORM", tiles)
    rng = np.random.default_rng(42700 + tiles)
    c, k = 72, 130
    x = rng.uniform(-1, 1, size=(1, 9, 15, c)).astype(np.float32)
    wt = (rng.uniform(0.1, 1, size=(k, 1, 1, c)) * rng.choice([-1, 1], size=(k, 1, 1, c))).astype(np.float32)
    x[0, 0, 0, 0] = np.inf
    x[0, 2, 1, 71] = -np.inf
    x[0, 2, 2, [3, 40]] = np.inf, -np.inf                # inf of either sign, or NaN
    x[0, 5, 7, 33] = np.nan
    x[0, 8, 14, 5] = np.finfo(np.float32).max            # one step below 2^128: bf16 rounds it up
    wt[77, 0, 0, 12] = -np.inf
    wt[129, 0, 0, 0] = 0.0                               # 0 * inf
    wt[3, 0, 0, 0] = 0.5                                 # pieces that are zero
    extra = rng.uniform(-1, 1, size=(1, 9, 15, k)).astype(np.float32)
    desc = G.make_desc(x.shape, wt.shape, (1, 1), (0, 0, 0, 0), 1)
    with np.errstate(all="ignore"):
        ref = (x.astype(np.float64)[0, :, :, None, :] * wt[None, None, :, 0, 0, :]).sum(axis=-1)[None] + (extra if add else 0)
    import torch
    import paper_1805_00907_amd as glowmi
    y = torch.from_numpy(extra).to("cuda:0") if add else G.poison(ref.shape, torch.float32)
    glowmi.conv2d_chain(G.dev(x), G.dev(wt), None, y, desc, addend=y if add else None, act=wl.ACT_NONE, workspace=None)
    torch.cuda.synchronize()
    assert glowmi.last_variant().startswith("conv_short_f32"), glowmi.last_variant()
    got = y.cpu().numpy()
    finite = np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[~finite & ~np.isnan(ref)], ref[~finite & ~np.isnan(ref)])
    mag = np.abs(np.where(np.isfinite(x), x, 0)).astype(np.float64)[0, :, :, None, :] * np.abs(np.where(np.isfinite(wt), wt, 0))[None, None, :, 0, 0, :]
    # 72 products of 24 bits: 73 roundings at most
    assert np.all(np.abs(got[finite] - ref[finite]) <= 73 * 2.0 ** -24 * (mag.sum(axis=-1)[None] + np.abs(extra))[finite])
