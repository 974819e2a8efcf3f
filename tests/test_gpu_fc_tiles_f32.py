"""fp32 FullyConnected cut on the way to the matrix cores (fc_tiles_f32) against the CPU oracle: ragged rows, columns and
reductions, fewer chunks than wavefronts, split reductions, values that outgrow a wavefront's scale (before and after sums have
been put aside), and what the kernels over fp16 pieces promise about accuracy, scales, zeros and non-finite values."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


SHAPES = [(1, 1, 1), (17, 16, 64), (33, 130, 65), (64, 1000, 96), (65, 259, 33), (138, 783, 223), (100, 513, 130), (130, 2048, 192)]


@pytest.mark.parametrize("rows", [32, 64])
@pytest.mark.parametrize("shape,split", [(s, 1) for s in SHAPES] + [(SHAPES[3], 3), (SHAPES[5], 3), (SHAPES[7], 2), (SHAPES[7], 8)], ids=str)
def test_fc_tiles_f32(shape, split, rows, knobs):
    import gpu_util as G
    m, k, n = shape
    knobs.set("F32_FC_TILES", 3 if rows == 32 else 4)
    knobs.set("F32_FC_TILES_SPLIT", split)
    rng = np.random.default_rng(39000 + m + k + n)
    a = rng.uniform(-1, 1, size=(m, k)).astype(np.float32)
    w = (rng.uniform(-1, 1, size=(k, n)) / np.sqrt(k)).astype(np.float32)
    a[:, :k // 2] /= 37.0                                # later chunks outgrow the first one's scale
    w[:k // 3] /= 5.0
    b = rng.uniform(-0.1, 0.1, size=(n,)).astype(np.float32)
    for bias, act in ((b, wl.ACT_RELU), (None, wl.ACT_NONE)):
        got, variant = G.gpu_fc_f32(a, w, bias, act)
        assert variant.startswith("fc_tiles_f32_%dx" % rows), variant
        G.assert_close_f32(got, oracle.fc_f32(a, w, bias, act=act), f"{shape} [{variant}]")


@pytest.mark.parametrize("rows", [32, 64])
def test_long_reductions_are_summed_in_short_runs(rows, knobs):
    """Error against 64-bit sums, a reduction of 576 steps of 16, 72 per wavefront.  Cutting the operands: a quarter of the
    values lose their last bit, 2^-24 rms of the value, twice.  An addition to an accumulator rounds by 0.29 of 2^-23 rms; n
    of them to a growing sum count as n / 2: runs of eight, nine runs, eight wavefronts.  (A run of 72 would give 2.4e-7.)"""
    import gpu_util as G
    knobs.set("F32_FC_TILES", 3 if rows == 32 else 4)
    knobs.set("F32_FC_TILES_SPLIT", 1)
    m, k, n = 64, 9216, 192
    rng = np.random.default_rng(39500)
    a = rng.standard_normal(size=(m, k)).astype(np.float32)
    w = (rng.standard_normal(size=(k, n)) / np.sqrt(k)).astype(np.float32)
    got, variant = G.gpu_fc_f32(a, w, None, wl.ACT_NONE)
    assert variant.startswith("fc_tiles_f32_%dx" % rows), variant
    ref = a.astype(np.float64) @ w.astype(np.float64)
    bound = 1.15 * np.sqrt(2 * 2.0 ** -48 + (0.29 * 2.0 ** -23) ** 2 * (8 / 2 + 9 / 2 + 8 / 2))
    assert np.linalg.norm(got - ref) <= bound * np.linalg.norm(ref), np.linalg.norm(got - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("shape,taken", [((64, 512, 256), False), ((65, 256, 64), True), ((1000, 1024, 512), True),
                                         ((256, 4096, 4096), True), ((150, 301, 77), True), ((1024, 4096, 4096), False)], ids=str)
def test_which_calls_take_the_kernel(shape, taken, knobs):
    """From 65 rows, up to where the contraction over planes is faster; only with the workspace the query names.  The call
    that works in the static buffer runs what the call with a workspace runs."""
    import torch
    import gpu_util as G
    import paper_1805_00907_amd as glowmi
    m, k, n = shape
    knobs.set("F32_FC_FEW", 0)               # which takes small matrices and few rows
    a, w = torch.randn((m, k), device="cuda:0"), torch.randn((k, n), device="cuda:0")
    y = G.poison((m, n), torch.float32)
    need = glowmi.fc_workspace_bytes(m, k, n)
    assert need > 0 or not taken

    def variant(workspace_bytes):
        ws = torch.empty(workspace_bytes, dtype=torch.uint8, device="cuda:0") if workspace_bytes else None
        glowmi.fc(a, w, None, y, m, k, n, wl.ACT_NONE, ws)
        return glowmi.last_variant()

    full = variant(need)
    assert full.startswith("fc_tiles_f32") == taken, full
    for too_small in (0, max(need - 1, 0)):
        assert not variant(too_small).startswith(("fc_tiles_f32", "igemm_f32_p3")), too_small
    if taken:
        try:
            glowmi.fc_noalloc(a, w, None, y, m, k, n)
            assert glowmi.last_variant() == full
        except glowmi.GlowmiError as e:
            assert e.status == 3 and "scratch" in str(e), e   # the limit is that of the fp32 kernel's partial sums
    torch.cuda.synchronize()


@pytest.mark.parametrize("shape", [(150, 301, 77), (256, 4096, 4096)], ids=str)
def test_switching_piece_contractions_off_covers_the_kernel(shape, knobs):
    import torch
    import gpu_util as G
    import paper_1805_00907_amd as glowmi
    m, k, n = shape
    knobs.set("F32_P3", 0)
    knobs.set("F32_FC_FEW", 0)
    a, w = torch.randn((m, k), device="cuda:0"), torch.randn((k, n), device="cuda:0")
    y = G.poison((m, n), torch.float32)
    glowmi.fc(a, w, None, y, m, k, n, wl.ACT_NONE, G.workspace(glowmi.fc_workspace_bytes(m, k, n)))
    assert glowmi.last_variant().startswith("igemm_f32_") and "p3" not in glowmi.last_variant(), glowmi.last_variant()
    if glowmi.fc_workspace_bytes(m, k, n) <= glowmi.fc_noalloc_max_scratch_bytes():
        glowmi.fc_noalloc(a, w, None, y, m, k, n)
        assert glowmi.last_variant().startswith("igemm_f32_") and "p3" not in glowmi.last_variant(), glowmi.last_variant()
    torch.cuda.synchronize()


# rows of a tile; sizes: one pass of the wavefronts, and deep enough that each puts its sums aside twice and more
FORMS = [(rows, m, k, n) for rows in (32, 64) for m, k, n in ((70, 133, 97), (33, 2500, 70))]


def _operands(seed, m, k, n):
    rng = np.random.default_rng(seed)
    a = rng.uniform(-1, 1, size=(m, k)).astype(np.float32)
    w = (rng.standard_normal(size=(k, n)) / np.sqrt(k)).astype(np.float32)
    return a, w, rng.uniform(-0.1, 0.1, size=(n,)).astype(np.float32), rng


def _run(rows, a, w, b, knobs):
    import gpu_util as G
    knobs.set("F32_FC_TILES", 3 if rows == 32 else 4)
    knobs.set("F32_FC_TILES_SPLIT", 1)
    got, variant = G.gpu_fc_f32(a, w, b, wl.ACT_NONE)
    assert variant.startswith("fc_tiles_f32_%dx" % rows), variant
    return got


def _exact_and_scale(a, w, b):
    a, w, b = (v.astype(np.float64) for v in (a, w, b))
    return a @ w + b, np.abs(a) @ np.abs(w) + np.abs(b)


@pytest.mark.parametrize("form", FORMS, ids=str)
@pytest.mark.parametrize("ex,ew", [(80, -90), (-100, 40), (100, -90), (-50, -50), (13, 0)])
def test_power_of_two_scaling_changes_only_the_scale(form, ex, ew, knobs):
    rows, m, k, n = form
    a, w, b, _ = _operands(39600, m, k, n)
    a[:, k // 2:] *= 64.0                                # the scale grows on the way
    base = _run(rows, a, w, b, knobs)
    got = _run(rows, np.ldexp(a, ex).astype(np.float32), np.ldexp(w, ew).astype(np.float32), np.ldexp(b, ex + ew).astype(np.float32),
               knobs)
    assert np.array_equal(np.ldexp(got.astype(np.float64), -(ex + ew)), base.astype(np.float64))


@pytest.mark.parametrize("form", FORMS, ids=str)
def test_wide_value_ranges_are_held_to_fp32_accuracy(form, knobs):
    """|gpu - exact| <= 4 * 2^-22 * (|A||W| + |b|): 24 binades of magnitudes in either operand and in both, and runs of the
    reduction of very different magnitude, growing and shrinking."""
    rows, m, k, n = form
    a, w, b, rng = _operands(39610, m, k, n)
    spread = lambda v: (v * np.exp2(rng.integers(-12, 13, size=v.shape))).astype(np.float32)
    steps = np.exp2(6.0 * (np.arange(k) * 5 // k)).astype(np.float32)      # within 2^28 of the largest
    cases = [(spread(a), w), (a, spread(w)), (spread(a), spread(w))]
    for order in (steps, steps[::-1], steps[rng.permutation(k)]):
        cases += [(a * order, w), (a, w * order[:, None]), (a * order, w * order[::-1][:, None])]
    for av, wv in cases:
        av[::7, ::5] = 0.0
        got = _run(rows, av, wv, b, knobs)
        exact, scale = _exact_and_scale(av, wv, b)
        assert np.all(np.isfinite(got))
        worst = float((np.abs(got - exact) / scale).max())
        assert worst <= 4 * 2.0 ** -22, worst


@pytest.mark.parametrize("form", FORMS, ids=str)
@pytest.mark.parametrize("where", ["input", "weight", "both"])
@pytest.mark.parametrize("last", [False, True])
def test_elements_far_below_the_largest(form, where, last, knobs):
    """One huge element, first or last in the reduction: the others are cut with what is left of them, an absolute error below
    2^-39 of the largest magnitude they are scaled by, and the product of two of them may be dropped."""
    rows, m, k, n = form
    a, w, b, _ = _operands(39620, m, k, n)
    at = k - 1 if last else 0
    if where in ("input", "both"):
        a[3, at] = np.float32(2.0 ** 33)
    if where in ("weight", "both"):
        w[at, 5] = np.float32(2.0 ** 31)
    got = _run(rows, a, w, b, knobs)
    exact, scale = _exact_and_scale(a, w, b)
    bound = 4 * 2.0 ** -22 * scale + 2.0 ** -38 * float(np.abs(a).max()) * float(np.abs(w).max()) * k
    assert np.all(np.isfinite(got)) and np.all(np.abs(got - exact) <= bound)
    if where != "both":
        assert float((np.abs(got - exact) / scale).max()) <= 2.0 ** -9


@pytest.mark.parametrize("form", FORMS, ids=str)
def test_zero_and_subnormal_operands(form, knobs):
    import gpu_util as G
    rows, m, k, n = form
    a, w, b, _ = _operands(39630, m, k, n)
    for az, wz in ((np.zeros_like(a), w), (a, np.zeros_like(w))):
        got = _run(rows, az, wz, b, knobs)
        assert np.array_equal(got, np.broadcast_to(b, got.shape))
    tiny = (a * np.float32(2.0 ** -140)).astype(np.float32)          # fp32 subnormals and zeros
    G.assert_close_f32(_run(rows, tiny, w, b, knobs), oracle.fc_f32(tiny, w, b, act=wl.ACT_NONE), "subnormal input")


@pytest.mark.parametrize("form", FORMS, ids=str)
@pytest.mark.parametrize("what", ["inf_in_input", "nan_in_input", "inf_in_weight", "nan_in_weight"])
@pytest.mark.parametrize("at", [0, -1])
def test_non_finite_operands_never_give_wrong_finite_values(form, what, at, knobs):
    """What a non-finite element reaches is not finite; other outputs are right or NaN; other rows' tiles are right.  (A tile of
    columns that ends inside the matrix also fetches columns of the next row.)"""
    rows, m, k, n = form
    a, w, b, _ = _operands(39640, m, k, n)
    value = np.inf if what.startswith("inf") else np.nan
    if what.endswith("input"):
        a[2, at] = value
    else:
        w[at, 3] = value
    got = _run(rows, a, w, b, knobs)
    ref = oracle.fc_f32(a, w, b, act=wl.ACT_NONE)
    reached = ~np.isfinite(ref)
    assert reached.any() and not np.isfinite(got[reached]).any()
    rest = ~reached & ~np.isnan(got)
    assert np.all(np.abs(got[rest] - ref[rest]) <= 1e-5 + 1e-4 * np.abs(ref[rest]))
    if what.endswith("input"):
        assert np.all(np.isfinite(got[rows:]))
