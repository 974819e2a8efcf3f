"""The int8 kernel for convolutions on few pixels with any reduction (conv_few_i8) through the C ABI against the CPU oracle, bit
for bit: every tile form, ragged pixels, channels and reductions, the last bytes of both tensors, taps on padding, filters
with an offset, both forms of the requantize step, with and without an addend."""
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
    (1, 1, 1, 1, 1, 1, 1, (1, 1), (0, 0, 0, 0)),
    (1, 5, 5, 12, 17, 3, 3, (1, 1), (1, 1, 1, 1)),         # chunks shorter than sixteen codes, channels that end inside four
    (2, 4, 4, 64, 16, 1, 1, (1, 1), (0, 0, 0, 0)),         # whole tiles, one step
    (2, 7, 9, 256, 40, 3, 3, (1, 1), (1, 1, 1, 1)),
    (1, 11, 6, 100, 33, 3, 3, (2, 1), (0, 1, 2, 1)),       # one-sided padding, a last chunk of four codes
    (3, 3, 3, 36, 66, 5, 4, (2, 2), (2, 3, 2, 2)),         # most taps on padding
    (1, 6, 6, 1032, 24, 1, 1, (1, 1), (0, 0, 0, 0)),
    (1, 3, 5, 520, 20, 3, 3, (1, 1), (1, 1, 1, 1)),        # several trips in every form
    (1, 9, 13, 24, 31, 1, 1, (2, 2), (0, 0, 0, 0)),
]


@pytest.mark.parametrize("tile", range(3))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:7])))
def test_conv_few_i8(shape, tile, knobs):
    G = _gpu()
    n, h, w, c, k, r, s, st, pd = shape
    knobs.set("I8_FEW", 2)
    knobs.set("I8_FEW_TILE", tile)
    rng = np.random.default_rng(39500 + c + k)
    x = rng.integers(-128, 128, size=(n, h, w, c), dtype=np.int8)
    wt = rng.integers(-128, 128, size=(k, r, s, c), dtype=np.int8)
    desc = G.make_desc(x.shape, wt.shape, st, pd, 1)
    for w_off, big, act in ((0, False, wl.ACT_RELU), (7, False, wl.ACT_NONE), (0, True, wl.ACT_NONE)):
        xs, ws = 0.031, 0.0043
        # the multiplier of the requantize step: as layers have it, or 0.7, which takes its 64-bit form
        ys = xs * ws / (0.7 if big else 0.01 / np.sqrt(r * s * c))
        qp = wl.QParams(xs, -9, ws, w_off, ys, 3)
        b = rng.integers(-3000, 3000, size=(k,), dtype=np.int32)
        args = (x, xs, -9, wt, ws, w_off, b)
        ref = oracle.qconv2d(*args, ys, 3, st, pd, 1, act=act)
        got, variant = G.gpu_qconv2d(x, wt, b, qp, desc, act)
        assert variant.startswith("conv_few_i8_16x"), variant
        G.assert_equal_i8(got, ref, f"{shape} w_off {w_off} [{variant}]")
        add = rng.integers(-128, 128, size=ref.shape, dtype=np.int8)
        ref = oracle.qconv2d_add(*args, add, 0.05, 11, ys, 3, st, pd, 1, act=act)
        for in_place in (False, True):
            got, variant = G.gpu_qconv2d_chain(x, wt, b, qp, add, 0.05, 11, desc, act, in_place=in_place)
            assert variant.startswith("conv_few_i8_16x"), variant
            G.assert_equal_i8(got, ref, f"{shape} add w_off {w_off} in place {in_place} [{variant}]")
