"""The int8 kernel for convolutions with a short reduction (conv_short_i8) through the C ABI against the CPU oracle, bit for bit:
every slice width, ragged pixels, channels and reductions, trips past the reduction, the last bytes of both tensors, taps on
padding, several blocks to a wavefront, every form of the requantize step, with and without an addend."""
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
    (1, 1, 1, 4, 4, 1, 1, (1, 1), (0, 0, 0, 0)),
    (1, 5, 5, 12, 20, 3, 3, (1, 1), (1, 1, 1, 1)),         # chunks of twelve codes, a run of four channels behind a whole one
    (2, 4, 4, 64, 32, 1, 1, (1, 1), (0, 0, 0, 0)),         # whole blocks, tiles and trips
    (2, 17, 9, 72, 136, 1, 1, (1, 1), (0, 0, 0, 0)),       # slices that end inside a tile
    (1, 11, 6, 100, 36, 2, 2, (2, 1), (0, 1, 2, 1)),       # one-sided padding, a last chunk of four codes
    (3, 3, 3, 36, 68, 3, 4, (2, 2), (2, 3, 2, 2)),         # most taps on padding
    (1, 6, 7, 520, 24, 1, 1, (1, 1), (0, 0, 0, 0)),        # several trips
    (1, 9, 13, 24, 28, 1, 1, (2, 2), (0, 0, 0, 0)),
    (1, 9, 13, 24, 28, 1, 1, (1, 1), (1, 0, 0, 2)),        # a single tap on padding
    (2, 7, 9, 128, 40, 1, 1, (1, 1), (0, 0, 0, 0)),        # rows whole cache lines apart, one trip
    (1, 6, 7, 128, 36, 2, 2, (1, 2), (1, 0, 0, 1)),        # the same, several trips, taps on padding
    (2, 5, 7, 1, 8, 1, 1, (1, 1), (0, 0, 0, 0)),           # channels at every byte of a dword, the last bytes of both tensors
    (1, 5, 6, 13, 24, 3, 3, (1, 1), (1, 1, 1, 1)),
    (3, 7, 5, 31, 36, 1, 1, (1, 1), (0, 0, 0, 0)),
    (1, 6, 9, 50, 132, 2, 3, (2, 1), (1, 0, 0, 2)),
    (1, 7, 8, 16, 132, 3, 3, (1, 1), (0, 0, 0, 0)),        # no padding
]


def _check(G, shape, rng, label, cases):
    n, h, w, c, k, r, s, st, pd = shape
    x = rng.integers(-128, 128, size=(n, h, w, c), dtype=np.int8)
    wt = rng.integers(-128, 128, size=(k, r, s, c), dtype=np.int8)
    desc = G.make_desc(x.shape, wt.shape, st, pd, 1)
    b = rng.integers(-3000, 3000, size=(k,), dtype=np.int32)
    for mult, act in cases:
        xs, ws = 0.031, 0.0043
        ys = xs * ws / (mult if mult else 0.01 / np.sqrt(r * s * c))
        qp = wl.QParams(xs, -9, ws, 0, ys, 3)
        args = (x, xs, -9, wt, ws, 0, b)
        ref = oracle.qconv2d(*args, ys, 3, st, pd, 1, act=act)
        got, variant = G.gpu_qconv2d(x, wt, b, qp, desc, act)
        assert variant.startswith("conv_short_i8"), variant
        G.assert_equal_i8(got, ref, f"{label} {mult} [{variant}]")
        add = rng.integers(-128, 128, size=ref.shape, dtype=np.int8)
        ref = oracle.qconv2d_add(*args, add, 0.05, 11, ys, 3, st, pd, 1, act=act)
        for in_place in (False, True):
            got, variant = G.gpu_qconv2d_chain(x, wt, b, qp, add, 0.05, 11, desc, act, in_place=in_place)
            assert variant.startswith("conv_short_i8"), variant
            G.assert_equal_i8(got, ref, f"{label} {mult} add in place {in_place} [{variant}]")


@pytest.mark.parametrize("tiles", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:7])) + "p" + "".join(map(str, s[8])))
def test_conv_short_i8(shape, tiles, knobs):
    knobs.set("I8_SHORT", 2)
    knobs.set("I8_SHORT_FORM", tiles)
    # the multiplier of the requantize step: as layers have it, 0.7 (its 64-bit form), and one whose offset does not fold
    _check(_gpu(), shape, np.random.default_rng(40500 + shape[3] + shape[4]), f"{shape} tiles {tiles}",
           ((0, wl.ACT_RELU), (0.7, wl.ACT_NONE), (2.0 ** -26, wl.ACT_NONE)))


# long reductions: the filter reaches LDS in passes of 64 chunks of 16 codes, each lane with one to four of them
# n  h  w  c  k  r  s  stride  pads, the slices (in tiles of 32 channels) whose filters LDS holds
LONG = [
    ((1, 7, 6, 92, 68, 3, 3, (1, 1), (1, 1, 1, 1)), (1, 2)),      # 54 chunks: one pass of four to a lane
    ((1, 4, 9, 796, 36, 1, 1, (1, 1), (0, 0, 0, 0)), (1, 2)),     # 50, a single tap
    ((2, 6, 7, 100, 40, 3, 3, (1, 1), (1, 1, 1, 1)), (1, 2)),     # 63 and zeros up to 66: a second pass of zeros but one
    ((1, 5, 4, 1021, 36, 1, 1, (1, 1), (0, 0, 0, 0)), (1, 2)),    # 64, the last one cut, channels at every byte of a dword
    ((2, 5, 6, 128, 72, 3, 3, (2, 1), (1, 1, 1, 1)), (1, 2)),     # 72, rows whole cache lines apart, a stride
    ((1, 5, 7, 125, 44, 3, 3, (1, 1), (1, 0, 2, 1)), (1, 2)),     # 72, channels at every byte, one-sided padding
    ((1, 4, 5, 1100, 36, 1, 1, (1, 1), (0, 0, 0, 0)), (1, 2)),    # 69 and zeros up to 72, a single tap
    ((2, 5, 6, 136, 40, 3, 3, (1, 1), (1, 1, 1, 1)), (1,)),       # 81 and zeros up to 84
    ((1, 4, 5, 228, 68, 3, 3, (1, 2), (1, 1, 1, 1)), (1,)),       # 135 and zeros up to 138: a third pass
    ((1, 4, 5, 231, 36, 3, 3, (1, 1), (1, 1, 1, 1)), (1,)),       # the same, channels at every byte
]


@pytest.mark.parametrize("shape,tiles", [(shape, t) for shape, forms in LONG for t in forms], ids=lambda v: "x".join(map(str, v[:7])) if isinstance(v, tuple) else str(v))
def test_conv_short_i8_long_reductions(shape, tiles, knobs):
    """Code sums, places in the image and zeros behind the reduction that go on from one pass of the filter's staging to the next."""
    knobs.set("I8_SHORT", 2)
    knobs.set("I8_SHORT_FORM", tiles)
    _check(_gpu(), shape, np.random.default_rng(40900 + shape[3] + shape[4]), f"{shape} tiles {tiles}", ((0, wl.ACT_RELU), (0.7, wl.ACT_NONE)))


@pytest.mark.parametrize("shape", [(3, 61, 77, 24, 40, 1, 1, (1, 1), (0, 0, 0, 0)), (2, 70, 53, 12, 136, 3, 3, (1, 1), (1, 1, 1, 1))],
                         ids=lambda s: "x".join(map(str, s[:7])))
def test_conv_short_i8_several_blocks(shape, knobs):
    """More blocks of pixels than wavefronts: slices of 32 channels of a layer of 34 leave few workgroups to each."""
    knobs.set("I8_SHORT", 2)
    knobs.set("I8_SHORT_FORM", 1)
    G = _gpu()
    n, h, w, c, k, r, s, st, pd = shape
    _check(G, (n, h, w, c, 34 * 32, r, s, st, pd), np.random.default_rng(40600 + c), f"{shape}", ((0, wl.ACT_RELU),))


def test_conv_short_i8_is_planned():
    """The planner's own choice, and what it leaves: filters with an offset."""
    G = _gpu()
    for c, k, w_off, taken in ((24, 208, 0, True), (24, 208, 5, False), (24, 206, 0, True), (23, 208, 0, True)):
        rng = np.random.default_rng(40700 + c + k + w_off)
        x = rng.integers(-128, 128, size=(2, 75, 70, c), dtype=np.int8)
        wt = rng.integers(-128, 128, size=(k, 3, 3, c), dtype=np.int8)
        qp = wl.QParams(0.03, 4, 0.004, w_off, 0.3, -2)
        ref = oracle.qconv2d(x, 0.03, 4, wt, 0.004, w_off, None, 0.3, -2, (1, 1), (1, 1, 1, 1), 1, act=wl.ACT_RELU)
        got, variant = G.gpu_qconv2d(x, wt, None, qp, G.make_desc(x.shape, wt.shape, (1, 1), (1, 1, 1, 1), 1), wl.ACT_RELU)
        assert variant.startswith("conv_short_i8") == taken, variant
        G.assert_equal_i8(got, ref, f"{c} {k} w_off {w_off} [{variant}]")


@pytest.mark.parametrize("tiles", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", [(1, 5, 7, 12, 1, 3, 3), (2, 6, 7, 33, 29, 1, 1), (1, 9, 8, 20, 131, 2, 2), (3, 5, 5, 64, 94, 1, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_conv_short_i8_odd_outputs(shape, tiles, knobs):
    """Pixels that start at any byte address; with an addend such a layer takes another kernel."""
    G = _gpu()
    knobs.set("I8_SHORT", 2)
    knobs.set("I8_SHORT_FORM", tiles)
    n, h, w, c, k, r, s = shape
    rng = np.random.default_rng(40800 + c + k)
    x = rng.integers(-128, 128, size=(n, h, w, c), dtype=np.int8)
    wt = rng.integers(-128, 128, size=(k, r, s, c), dtype=np.int8)
    b = rng.integers(-3000, 3000, size=(k,), dtype=np.int32)
    pd = (r // 2,) * 4
    qp = wl.QParams(0.03, 4, 0.004, 0, 0.3, -2)
    desc = G.make_desc(x.shape, wt.shape, (1, 1), pd, 1)
    args = (x, 0.03, 4, wt, 0.004, 0, b)
    ref = oracle.qconv2d(*args, 0.3, -2, (1, 1), pd, 1, act=wl.ACT_RELU)
    got, variant = G.gpu_qconv2d(x, wt, b, qp, desc, wl.ACT_RELU)
    assert variant.startswith("conv_short_i8"), variant
    G.assert_equal_i8(got, ref, f"{shape} tiles {tiles} [{variant}]")
    add = rng.integers(-128, 128, size=ref.shape, dtype=np.int8)
    ref = oracle.qconv2d_add(*args, add, 0.05, 11, 0.3, -2, (1, 1), pd, 1, act=wl.ACT_NONE)
    got, variant = G.gpu_qconv2d_chain(x, wt, b, qp, add, 0.05, 11, desc, wl.ACT_NONE)
    assert not variant.startswith("conv_short_i8") or k % 4 == 0, variant
    G.assert_equal_i8(got, ref, f"{shape} add [{variant}]")
