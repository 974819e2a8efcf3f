"""fp32 FullyConnected cut on the way to the matrix cores (fc_tiles_f32) against the CPU oracle: ragged rows, columns and
reductions, fewer chunks than wavefronts, split reductions, values that outgrow a wavefront's scale."""
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
def test_which_calls_take_the_kernel(shape, taken):
    """From 65 rows, up to where the contraction over planes is faster; only with the workspace the query names.  The call
    that works in the static buffer runs what the call with a workspace runs."""
    import torch
    import gpu_util as G
    import paper_1805_00907_amd as glowmi
    m, k, n = shape
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
    a, w = torch.randn((m, k), device="cuda:0"), torch.randn((k, n), device="cuda:0")
    y = G.poison((m, n), torch.float32)
    glowmi.fc(a, w, None, y, m, k, n, wl.ACT_NONE, G.workspace(glowmi.fc_workspace_bytes(m, k, n)))
    assert glowmi.last_variant().startswith("igemm_f32_") and "p3" not in glowmi.last_variant(), glowmi.last_variant()
    if glowmi.fc_workspace_bytes(m, k, n) <= glowmi.fc_noalloc_max_scratch_bytes():
        glowmi.fc_noalloc(a, w, None, y, m, k, n)
        assert glowmi.last_variant().startswith("igemm_f32_") and "p3" not in glowmi.last_variant(), glowmi.last_variant()
    torch.cuda.synchronize()
