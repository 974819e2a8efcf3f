"""The first layer on the fp16 matrix cores against the CPU oracle: every place that an aligned group of four of an image's row can
have in a patch (left padding 0 to 3), rows of every length modulo four, channel counts that end inside a store, both slice
widths, more tiles than workgroups, and the number of tiles from which the planner takes it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


def _gpu():
    import gpu_util
    return gpu_util


def _check(G, n, h, w, k, pads):
    rng = np.random.default_rng(41000 + h + w + k)
    x = rng.uniform(-1, 1, size=(n, h, w, 3)).astype(np.float32)
    wt = (rng.uniform(-1, 1, size=(k, 7, 7, 3)) / 12).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(k,)).astype(np.float32)
    ref = oracle.conv2d_f32(x, wt, b, (2, 2), pads, 1, act=wl.ACT_NONE)
    got, variant = G.gpu_conv2d_f32(x, wt, b, G.make_desc(x.shape, wt.shape, (2, 2), pads, 1), wl.ACT_NONE)
    G.assert_close_f32(got, ref, f"{n}x{h}x{w} k {k} pads {pads} [{variant}]")
    return variant


@pytest.mark.parametrize("pad_l", [0, 1, 2, 3])
@pytest.mark.parametrize("w", [36, 37, 38, 39])
@pytest.mark.parametrize("k", [8, 61, 98])
def test_first_layer_f16_patches(pad_l, w, k, knobs):
    knobs.set("F32_SMALLC_BF16", 1)
    assert _check(_gpu(), 2, 23, w, k, (3, pad_l, 1, 3 - pad_l)).endswith("f16x3")


def test_first_layer_f16_many_tiles(knobs):
    knobs.set("F32_SMALLC_BF16", 1)
    assert _check(_gpu(), 31, 46, 101, 40, (3, 3, 3, 3)).endswith("f16x3")   # 930 tall tiles to a slice of 32 channels


@pytest.mark.parametrize("n,taken", [(5, False), (6, True)])
def test_first_layer_f16_is_planned(n, taken):
    """A map of 50 tiles of 4 x 16 pixels."""
    assert _check(_gpu(), n, 80, 160, 64, (3, 3, 3, 3)).endswith("f16x3") == taken


@pytest.mark.parametrize("n,k", [(1, 64), (5, 64), (3, 128), (2, 192), (4, 96), (1, 330)])
def test_first_layer_below_300_tiles_keeps_every_bit(n, k):
    """The same map, filters of one tap: below 300 tiles the product is one of fp32 operands and gives the input back bit for bit, whatever
    the number of channels (two fp16 pieces hold 22 of the 24 bits)."""
    G = _gpu()
    rng = np.random.default_rng(41300 + n + k)
    x = rng.uniform(-1, 1, size=(n, 80, 160, 3)).astype(np.float32)
    taps = rng.integers(0, [7, 7, 3], size=(k, 3))
    wt = np.zeros((k, 7, 7, 3), np.float32)
    wt[np.arange(k), taps[:, 0], taps[:, 1], taps[:, 2]] = 1
    got, variant = G.gpu_conv2d_f32(x, wt, None, G.make_desc(x.shape, wt.shape, (2, 2), (3, 3, 3, 3), 1), wl.ACT_NONE)
    assert variant.startswith("conv_smallc_f32"), variant
    padded = np.pad(x, ((0, 0), (3, 3), (3, 3), (0, 0)))
    for i, (r, s, c) in enumerate(taps):
        assert np.array_equal(got[..., i], padded[:, r:r + 80:2, s:s + 160:2, c]), (i, variant)


@pytest.mark.parametrize("place", ["input", "filter"])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_first_layer_f16_non_finite(place, value, knobs):
    """A value that no scale fits: the outputs it reaches are what fp32 arithmetic gives, all others as close as ever, those of its
    tile and of the tiles that its workgroup takes later among them."""
    G = _gpu()
    knobs.set("F32_SMALLC_BF16", 1)
    rng = np.random.default_rng(41500)
    x = rng.uniform(-1, 1, size=(31, 46, 101, 3)).astype(np.float32)
    wt = (rng.uniform(0.1, 1, size=(40, 7, 7, 3)) / 12).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(40,)).astype(np.float32)
    if place == "input":
        x[0, 0, 0, 1] = x[2, 20, 50, 2] = x[30, 45, 100, 0] = value
    else:
        wt[17, 3, 2, 1] = value
    ref = oracle.conv2d_f32(x, wt, b, (2, 2), (3, 3, 3, 3), 1, act=wl.ACT_NONE)
    got, variant = G.gpu_conv2d_f32(x, wt, b, G.make_desc(x.shape, wt.shape, (2, 2), (3, 3, 3, 3), 1), wl.ACT_NONE)
    assert variant.endswith("f16x3")
    finite = np.isfinite(ref)
    assert 0 < (~finite).sum() < ref.size // 30
    assert np.array_equal(got[~finite], ref[~finite], equal_nan=True)
    G.assert_close_f32(np.where(finite, got, 0), np.where(finite, ref, 0), f"{place} {value}")
