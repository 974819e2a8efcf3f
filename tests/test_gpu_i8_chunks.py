"""int8 convolutions and FullyConnected layers whose channel counts, reductions and columns fit no 16-byte chunk: the kernels
that walk the reduction in 16-code chunks (igemm_i8, conv_small_i8) and the strip form of fc_small_i8, against the oracle
bit for bit.  The last pixel, filter and weight row end exactly at the end of their tensors, so the loads that would run
past it are the shifted ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


def _gpu():
    import gpu_util
    return gpu_util


# n  h   w   c    k    r  stride pad groups
CONVS = [
    (1, 5, 7, 1, 1, 1, 1, 0, 1),          # one code per chunk, one output channel
    (2, 9, 8, 3, 5, 3, 2, 1, 1),
    (1, 7, 7, 15, 33, 3, 1, 1, 1),        # one code short of a chunk; a channel tile of one
    (1, 6, 11, 17, 31, 3, 1, 1, 1),       # two chunks per tap, the second of one code
    (3, 13, 9, 72, 120, 3, 1, 1, 1),
    (1, 12, 12, 61, 66, 5, 2, 2, 1),
    (2, 8, 8, 40, 24, 3, 1, 1, 2),        # groups: 20 codes per tap, the neighbouring group's channels behind them
    (1, 4, 4, 2056, 12, 1, 1, 0, 1),      # deep pointwise reduction: the slices over the grid
    (2, 17, 19, 50, 70, 1, 2, 0, 1),
]


@pytest.mark.parametrize("shape", CONVS, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("x_off,w_off", [(-9, 0), (13, -5)])
@pytest.mark.parametrize("kernel", ["small", "tile0", "tile6", "tile7"])
def test_qconv_any_channel_count(shape, x_off, w_off, kernel, knobs):
    G = _gpu()
    n, h, w, c, k, r, st, pd, g = shape
    if kernel == "small":
        knobs.set("I8_SMALL_MAX_TILES", 100000)
    else:
        knobs.set("I8_TILE", kernel[4:])
    layer = wl.ConvLayer("chunks", n, h, w, c, k, r, r, st, pd, g)
    xq, wq, bq, qp = wl.conv_inputs_q(layer, 9100 + c + k, dist="uniform", w_off=w_off)
    qp = wl.QParams(qp.x_scale, x_off, qp.w_scale, w_off, qp.y_scale, qp.y_off)
    rq, r_scale, r_off = wl.addend_q(layer, 9100, qp.y_scale)
    desc = G.desc_of(layer)
    args = (xq, qp.x_scale, qp.x_off, wq, qp.w_scale, qp.w_off, bq)
    for use_ws in (True, False):
        ref = oracle.qconv2d(*args, qp.y_scale, qp.y_off, (st, st), (pd,) * 4, g, act=wl.ACT_RELU)
        got, variant = G.gpu_qconv2d(xq, wq, bq, qp, desc, wl.ACT_RELU, use_workspace=use_ws)
        G.assert_equal_i8(got, ref, f"{shape} {kernel} ws {use_ws} [{variant}]")
        ref = oracle.qconv2d_add(*args, rq, r_scale, r_off, qp.y_scale, qp.y_off, (st, st), (pd,) * 4, g, act=wl.ACT_RELU)
        got, variant = G.gpu_qconv2d_chain(xq, wq, bq, qp, rq, r_scale, r_off, desc, wl.ACT_RELU, use_workspace=use_ws)
        G.assert_equal_i8(got, ref, f"{shape} {kernel} add ws {use_ws} [{variant}]")
    if kernel == "small":
        assert variant.startswith("conv_small_i8") or c == 2056, variant


# n  h   w  c  k   r  s  pads (t, l, b, r): the codes within three bytes of a tensor's end belong to a pixel (or filter) that is
# the last of a tile of 32, 64 or 128, with another tile behind it
NEAR_END = [(m, 1, 1, 1, 20, 1, 1, (0, 0, 0, 0)) for m in (33, 34, 35, 65, 66, 67, 129, 130, 131)] + \
           [(1, m + 2, 1, 1, 20, 3, 1, (0, 0, 2, 0)) for m in (32, 34, 64, 66, 130)] + \
           [(1, 17, 2, 1, 20, 1, 1, (0, 0, 0, 0)), (17, 1, 2, 1, 20, 1, 1, (0, 0, 0, 0)), (11, 3, 1, 2, 9, 2, 1, (0, 0, 3, 0))] + \
           [(1, 11, 13, 1, k, 1, 1, (0, 0, 0, 0)) for k in (33, 34, 35, 65, 66, 67, 129, 130)] + \
           [(1, 11, 13, 2, 34, 1, 1, (0, 0, 0, 0)), (1, 12, 13, 1, 33, 2, 1, (0, 0, 0, 0))]


@pytest.mark.parametrize("shape", NEAR_END, ids=lambda s: "x".join(map(str, s[:7])) + "p%d" % s[7][2])
@pytest.mark.parametrize("kernel", ["small", "tile0", "tile2"])
@pytest.mark.parametrize("w_off", [0, 6])
def test_qconv_codes_at_the_end_of_a_tensor(shape, kernel, w_off, knobs):
    G = _gpu()
    n, h, w, c, k, r, s, pads = shape
    if kernel == "small":
        knobs.set("I8_SMALL_MAX_TILES", 100000)
    else:
        knobs.set("I8_TILE", kernel[4:])
    rng = np.random.default_rng(9150 + n + h + k)
    xq = rng.integers(-128, 128, size=(n, h, w, c)).astype(np.int8)
    wq = rng.integers(-128, 128, size=(k, r, s, c)).astype(np.int8)
    qp = wl.QParams(0.05, -9, 0.04, w_off, 0.9, 3)
    ref = oracle.qconv2d(xq, qp.x_scale, qp.x_off, wq, qp.w_scale, qp.w_off, None, qp.y_scale, qp.y_off, (1, 1), pads, 1,
                         act=wl.ACT_NONE)
    got, variant = G.gpu_qconv2d(xq, wq, None, qp, G.make_desc(xq.shape, wq.shape, (1, 1), pads, 1), wl.ACT_NONE)
    assert variant.startswith("conv_small_i8" if kernel == "small" else "igemm_i8"), variant
    G.assert_equal_i8(got, ref, f"{shape} {kernel} [{variant}]")


@pytest.mark.parametrize("m,k", [(m, k) for m in (33, 34, 35, 36, 65, 66, 67, 68) for k in (1, 2, 17)])
@pytest.mark.parametrize("kernel", ["strip", "tile0"])
def test_qfc_codes_at_the_end_of_the_activations(m, k, kernel, knobs):
    G = _gpu()
    if kernel != "strip":
        knobs.set("I8_TILE", 0)
    aq, wq, bq, qp = wl.fc_inputs_q(wl.FcLayer("end", m, k, 40), 9250 + m + k, dist="uniform", w_off=5)
    ref = oracle.qfc(aq, qp.x_scale, qp.x_off, wq, qp.w_scale, qp.w_off, bq, qp.y_scale, qp.y_off, act=wl.ACT_NONE)
    got, variant = G.gpu_qfc(aq, wq, bq, qp, wl.ACT_NONE)
    assert variant == ("fc_strip_i8" if kernel == "strip" else "igemm_i8_64x64w4_fc"), variant
    G.assert_equal_i8(got, ref, f"qfc {m}x{k} [{variant}]")


@pytest.mark.parametrize("shape", [(1, 17, 5), (33, 40, 36), (76, 808, 208), (65, 255, 33), (40, 1030, 50), (97, 2047, 7), (8, 300, 1)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("w_off", [0, 6])
def test_qfc_any_size(shape, w_off):
    G = _gpu()
    M, K, N = shape
    aq, wq, bq, qp = wl.fc_inputs_q(wl.FcLayer("strip", M, K, N), 9200 + M + K, dist="uniform", w_off=w_off)
    ref = oracle.qfc(aq, qp.x_scale, qp.x_off, wq, qp.w_scale, qp.w_off, bq, qp.y_scale, qp.y_off, act=wl.ACT_RELU)
    got, variant = G.gpu_qfc(aq, wq, bq, qp, wl.ACT_RELU)
    assert variant == "fc_strip_i8", variant
    G.assert_equal_i8(got, ref, f"qfc {shape} w_off {w_off}")
