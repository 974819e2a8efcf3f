"""The fp32 convolution kernel for layers of ordinary size (conv_patch_f32: 1x1 and 3x3, stride 1 or 2, fp16 piece products)
through the C ABI against the CPU oracle, element by element, |gpu - oracle| <= 1e-5 + 1e-4 |oracle|: every tile form on
maps, channel counts and strides that leave it ragged, with and without the add link, plain and with the filter's planes
made ahead of time; componentwise accuracy over 24 binades, chunks of very different magnitude in either order, and
non-finite inputs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


def _gpu():
    import gpu_util
    return gpu_util


# n  h   w   c    k   r  stride pad
SHAPES = [
    (1, 8, 8, 8, 8, 3, 1, 1),          # one tile, one short chunk
    (2, 9, 13, 40, 24, 3, 1, 1),       # ragged tiles, a chunk of eight channels behind a whole one
    (1, 7, 7, 96, 72, 3, 1, 1),        # a map smaller than a tile, channel tile of eight
    (3, 15, 10, 64, 130, 3, 1, 0),     # no padding, channel tiles of two
    (1, 33, 21, 32, 64, 3, 1, 1),
    (2, 16, 16, 64, 64, 3, 2, 1),      # stride 2
    (1, 13, 17, 72, 40, 3, 2, 1),
    (1, 9, 64, 32, 32, 3, 2, 1),
    (2, 9, 7, 13, 20, 3, 1, 1),        # channels that end inside a piece of eight, also behind a whole chunk
    (1, 12, 10, 65, 33, 3, 2, 1),
    (2, 7, 11, 131, 50, 1, 1, 0),
    (1, 5, 9, 3, 16, 1, 2, 0),
    (2, 11, 9, 64, 100, 1, 1, 0),      # pointwise: the last tile's pixels end inside it
    (1, 5, 5, 264, 40, 1, 1, 0),
    (3, 14, 11, 72, 136, 1, 2, 0),     # pointwise, stride 2
    (1, 3, 70, 8, 33, 1, 2, 0),
]


def _inputs(seed, n, h, w, c, k, r):
    rng = np.random.default_rng(seed)
    x = rng.uniform(-1, 1, size=(n, h, w, c)).astype(np.float32)
    wt = (rng.standard_normal(size=(k, r, r, c)) / np.sqrt(r * r * c)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(k,)).astype(np.float32)
    return x, wt, b, rng


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("tile", range(7))
def test_conv_patch(shape, tile, knobs):
    import torch
    import paper_1805_00907_amd as glowmi
    G = _gpu()
    n, h, w, c, k, r, st, pd = shape
    if (tile == 1 and r == 1) or (tile != 1 and (r, st) == (3, 2)):
        pytest.skip("no such form")
    knobs.set("F32_PATCH", 2)
    knobs.set("F32_PATCH_TILE", tile)
    knobs.set("F32_K3", 0)
    knobs.set("F32_K3C64", 0)
    x, wt, b, rng = _inputs(37000 + c + k, n, h, w, c, k, r)
    desc = G.make_desc(x.shape, wt.shape, (st, st), (pd,) * 4, 1)
    ref = oracle.conv2d_f32(x, wt, b, (st, st), (pd,) * 4, 1, act=wl.ACT_RELU)
    got, variant = G.gpu_conv2d_f32(x, wt, b, desc, wl.ACT_RELU)
    assert variant.startswith("conv_patch_f32_f16x3"), variant
    G.assert_close_f32(got, ref, f"{shape} [{variant}]")
    add = rng.uniform(-1, 1, size=ref.shape).astype(np.float32)
    ref = oracle.conv2d_f32_add(x, wt, None, add, (st, st), (pd,) * 4, 1, act=wl.ACT_NONE)
    for in_place in (False, True):
        got, variant = G.gpu_conv2d_f32_chain(x, wt, None, add, desc, wl.ACT_NONE, in_place=in_place)
        assert variant.startswith("conv_patch_f32_f16x3") and variant.endswith("_add"), variant
        G.assert_close_f32(got, ref, f"{shape} add [{variant}]")
    if c % 8:
        return                                          # no plane form
    planes = torch.empty(glowmi.conv2d_filter_planes_bytes(desc), dtype=torch.uint8, device="cuda:0")
    wd = G.dev(wt)
    glowmi.conv2d_pack_filter(wd, desc, planes)
    y = G.poison(ref.shape, torch.float32)
    ws = torch.empty(glowmi.conv2d_packed_workspace_bytes(desc), dtype=torch.uint8, device="cuda:0")
    glowmi.conv2d_packed(G.dev(x), wd, planes, None, y, desc, addend=G.dev(add), act=wl.ACT_NONE, workspace=ws)
    torch.cuda.synchronize()
    assert glowmi.last_variant() == variant
    G.assert_close_f32(y.cpu().numpy(), ref, f"{shape} packed [{variant}]")


@pytest.mark.parametrize("r,st", [(3, 1), (3, 2), (1, 1)])
def test_conv_patch_wide_value_ranges(r, st, knobs):
    G = _gpu()
    knobs.set("F32_PATCH", 2)
    knobs.set("F32_K3", 0)
    knobs.set("F32_K3C64", 0)
    n, h, w, c, k, pd = 2, 12, 12, 160, 40, r // 2
    x, wt, b, rng = _inputs(37500 + r + st, n, h, w, c, k, r)
    desc = G.make_desc(x.shape, wt.shape, (st, st), (pd,) * 4, 1)

    def bound(xv, wv):
        mag = oracle.conv2d_f32(np.abs(xv), np.abs(wv), np.abs(b), (st, st), (pd,) * 4, 1)
        return 4 * 2.0 ** -22 * mag.astype(np.float64)

    # 24 binades of magnitudes in both operands
    xs = (x * np.exp2(rng.integers(-12, 13, size=x.shape))).astype(np.float32)
    ws = (wt * np.exp2(rng.integers(-12, 13, size=wt.shape))).astype(np.float32)
    for xv, wv in ((xs, wt), (x, ws), (xs, ws)):
        ref = oracle.conv2d_f32(xv, wv, b, (st, st), (pd,) * 4, 1)
        got, variant = G.gpu_conv2d_f32(xv, wv, b, desc, wl.ACT_NONE)
        assert variant.startswith("conv_patch_f32_f16x3"), variant
        assert np.all(np.abs(got.astype(np.float64) - ref) <= bound(xv, wv) + 1e-30), variant
    # channel groups of very different magnitude, growing and shrinking: the accumulators are scaled along
    for order in (1, -1):
        xv = (x * np.exp2(order * 20.0 * (np.arange(c) // 32)).astype(np.float32)[None, None, None, :]).astype(np.float32)
        ref = oracle.conv2d_f32(xv, wt, b, (st, st), (pd,) * 4, 1)
        got, variant = G.gpu_conv2d_f32(xv, wt, b, desc, wl.ACT_NONE)
        assert np.all(np.abs(got.astype(np.float64) - ref) <= bound(xv, wt) + 1e-30), (order, variant)
    # zeros, and non-finite values: what they reach is not finite, nothing is finite and wrong
    got, _ = G.gpu_conv2d_f32(np.zeros_like(x), wt, b, desc, wl.ACT_NONE)
    assert np.array_equal(got, np.broadcast_to(b, got.shape))
    xv = x.copy()
    xv[1, 5, 5, 3] = np.inf
    xv[0, 2, 2, 40] = np.nan
    ref = oracle.conv2d_f32(xv, wt, b, (st, st), (pd,) * 4, 1)
    got, _ = G.gpu_conv2d_f32(xv, wt, b, desc, wl.ACT_NONE)
    reached = ~np.isfinite(ref)
    assert reached.any() and not np.isfinite(got[reached]).any()
    ok = np.isfinite(got)
    assert np.all(np.abs(got[ok].astype(np.float64) - ref[ok]) <= 1e-5 + 1e-4 * np.abs(ref[ok]))


@pytest.mark.parametrize("c", [13, 67])
@pytest.mark.parametrize("r,st", [(3, 1), (3, 2), (1, 1), (1, 2)])
def test_non_finite_values_with_channels_that_end_inside_a_piece(c, r, st, knobs):
    """A pixel's last piece of eight channels ends in the next pixel, whose values meet zeros of the filter: outputs that a
    non-finite one does not reach are right or NaN, never finite and wrong."""
    G = _gpu()
    knobs.set("F32_PATCH", 2)
    n, h, w, k = 2, 9, 11, 24
    x, wt, b, _ = _inputs(37600 + c, n, h, w, c, k, r)
    x[0, 4, 4, 0], x[0, 8, 2, 1], x[1, 2, 6, 0] = np.nan, -np.inf, np.inf
    desc = G.make_desc(x.shape, wt.shape, (st, st), (r // 2,) * 4, 1)
    ref = oracle.conv2d_f32(x, wt, b, (st, st), (r // 2,) * 4, 1, act=wl.ACT_NONE)
    got, variant = G.gpu_conv2d_f32(x, wt, b, desc, wl.ACT_NONE)
    assert variant.startswith("conv_patch_f32_f16x3"), variant
    reached = ~np.isfinite(ref)
    assert reached.any() and not np.isfinite(got[reached]).any()
    rest = ~reached & ~np.isnan(got)
    assert np.all(np.abs(got[rest] - ref[rest]) <= 1e-5 + 1e-4 * np.abs(ref[rest]))


@pytest.mark.parametrize("r,st,tile", [(r, st, t) for r, st in ((3, 1), (3, 2), (1, 1)) for t in range(7)
                                       if not (t == 1 and r == 1) and not (t != 1 and (r, st) == (3, 2))])
def test_long_reductions_are_summed_in_short_runs(r, st, tile, knobs):
    """Error against 64-bit sums of a reduction of 256 to 288 steps of 16.  Cutting the operands: a quarter of the values
    lose their last bit, 2^-24 rms of the value, twice.  An addition to an accumulator rounds by 0.29 of 2^-23 rms; n of them
    to a growing sum count as n / 2: runs of nine, then 32 runs.  (One run of 288 would give 4.2e-7.)"""
    G = _gpu()
    knobs.set("F32_PATCH", 2)
    knobs.set("F32_PATCH_TILE", tile)
    knobs.set("F32_K3", 0)
    knobs.set("F32_K3C64", 0)
    c = 512 if r == 3 else 4096
    rng = np.random.default_rng(37700)
    x = rng.standard_normal(size=(1, 16, 8, c)).astype(np.float32)
    wt = (rng.standard_normal(size=(64, r, r, c)) / np.sqrt(r * r * c)).astype(np.float32)
    desc = G.make_desc(x.shape, wt.shape, (st, st), (r // 2,) * 4, 1)
    ref = oracle.conv2d_f32(x, wt, None, (st, st), (r // 2,) * 4, 1, act=wl.ACT_NONE).astype(np.float64)
    got, variant = G.gpu_conv2d_f32(x, wt, None, desc, wl.ACT_NONE)
    assert variant.startswith("conv_patch_f32_f16x3"), variant
    bound = 1.15 * np.sqrt(2 * 2.0 ** -48 + (0.29 * 2.0 ** -23) ** 2 * (9 / 2 + 32 / 2))
    assert np.linalg.norm(got - ref) <= bound * np.linalg.norm(ref), np.linalg.norm(got - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("n,hw,c,k,st", [(16, 56, 128, 128, 2), (32, 7, 512, 512, 1), (8, 28, 128, 128, 1)])
def test_a_workspace_that_holds_the_cut_filter_is_enough(n, hw, c, k, st):
    """The query names more where the contraction over planes would run otherwise; a byte less than the cut filter and the
    workspace is left alone."""
    import torch
    import paper_1805_00907_amd as glowmi
    G = _gpu()
    desc = glowmi.ConvDesc(n, hw, hw, c, k, 3, 3, st, st, 1, 1, 1, 1, 1)
    x, w = torch.randn((n, hw, hw, c), device="cuda:0"), torch.randn((k, 3, 3, c), device="cuda:0")
    oh, ow = glowmi.conv_out_shape(desc)
    need = 4 * k * 9 * c + 4 * k                         # (a multiple of 256 here)
    assert glowmi.conv2d_workspace_bytes(desc) >= need
    out = []
    for given in (glowmi.conv2d_workspace_bytes(desc), need, need - 1):
        y = G.poison((n, oh, ow, k), torch.float32)
        ws = torch.full((given,), 0x5A, dtype=torch.uint8, device="cuda:0")
        glowmi.conv2d(x, w, None, y, desc, wl.ACT_NONE, ws)
        torch.cuda.synchronize()
        out.append((glowmi.last_variant(), y, bool((ws == 0x5A).all())))
    assert out[0][0].startswith("conv_patch_f32") and out[1][0] == out[0][0], (out[0][0], out[1][0])
    assert torch.equal(out[0][1], out[1][1])
    assert not out[2][0].startswith("conv_patch_f32") and out[2][2]


@pytest.mark.parametrize("layers", [1, 8, 10])
def test_sequence_cuts_filters_ahead_in_groups(layers, knobs):
    """Layers of a sequence have their filters cut up to eight at a time: the same results as layer by layer."""
    import torch
    import paper_1805_00907_amd as glowmi
    G = _gpu()
    knobs.set("F32_PATCH", 2)
    rng = np.random.default_rng(37900 + layers)
    widths = [24, 40, 16, 72, 8, 32, 136, 24, 64, 48, 24]
    x = rng.uniform(-1, 1, size=(2, 9, 11, widths[0])).astype(np.float32)
    seq, keep, step = [], [], G.dev(x)
    for i in range(layers):
        r, c, k = 3 if i % 2 else 1, widths[i], widths[i + 1]
        wd = G.dev((rng.standard_normal(size=(k, r, r, c)) / np.sqrt(r * r * c)).astype(np.float32))
        bd = G.dev(rng.uniform(-0.1, 0.1, size=(k,)).astype(np.float32))
        desc = G.make_desc(tuple(step.shape), (k, r, r, c), (1, 1), (r // 2,) * 4, 1)
        seq.append((desc, wd, bd, wl.ACT_RELU, False))
        y = torch.empty((2, 9, 11, k), device="cuda:0")
        ws = torch.empty(max(glowmi.conv2d_workspace_bytes(desc), 16), dtype=torch.uint8, device="cuda:0")
        glowmi.conv2d(step, wd, bd, y, desc, wl.ACT_RELU, ws)
        assert glowmi.last_variant().startswith("conv_patch_f32"), glowmi.last_variant()
        keep += [wd, bd, ws]
        step = y
    arr = glowmi.seq_layers(seq)
    arena = torch.empty(glowmi.seq_arena_bytes(arr, False), dtype=torch.uint8, device="cuda:0")
    got = G.poison(tuple(step.shape), torch.float32)
    for _ in range(2):
        glowmi.seq_conv2d(G.dev(x), arr, got, arena)
    torch.cuda.synchronize()
    assert torch.equal(got, step)
