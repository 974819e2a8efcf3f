"""fp32 FullyConnected over planes (igemm_f32_p3_fc) at the edges of its tiles and slabs.

Against the CPU oracle at |gpu - oracle| <= 1e-5 + 1e-4 |oracle|: one slab more and less than a workgroup folds its sums after
(16 slabs of 64), rows and columns one over a tile, a column count that takes single stores, more rows than have a scale each
(1024), and the weights' planes in the order the FullyConnected call makes them in as well as the one a convolution's are in (by
channel, a scale each), which the kernel has to notice.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl

# M, K, N, split (0: the planner's)
CASES = [(128, 1024, 128, 1), (129, 1032, 132, 1), (257, 2120, 65, 1), (130, 4104, 260, 2), (1100, 136, 136, 1), (33, 8, 1000, 0)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("order", ["rows", "by_channel", "cut_in_the_call"])
def test_fc_over_planes(case, order, knobs):
    import gpu_util as G
    import torch
    import paper_1805_00907_amd as glowmi
    M, K, N, split = case
    knobs.set("F32_P3_MIN_M", 1)
    knobs.set("F32_P3_RATIO", 0)
    if split:
        knobs.set("F32_SPLIT", split)
    a, w, b = wl.fc_inputs_f32(wl.FcLayer("planes", M, K, N), 47000 + M + K + N, dist="uniform_fan_in")
    a[::3] *= np.float32(2.0 ** 20)                                    # rows far apart
    ref = oracle.fc_f32(a, w, b, act=wl.ACT_RELU)
    ad, wd, bd = G.dev(a), G.dev(w), G.dev(b)
    whole, y = G.guarded((M, N), torch.float32)
    if order == "cut_in_the_call":
        glowmi.fc(ad, wd, bd, y, M, K, N, wl.ACT_RELU, G.workspace(glowmi.fc_workspace_bytes(M, K, N)))
    else:
        planes = torch.empty(glowmi.fc_filter_planes_bytes(K, N), dtype=torch.uint8, device="cuda:0")
        if order == "rows":
            glowmi.fc_pack_filter(wd, K, N, planes)
        else:
            desc = glowmi.ConvDesc(1, 8, 8, K, N, 1, 1, 1, 1, 0, 0, 0, 0, 1)
            assert glowmi.conv2d_filter_planes_bytes(desc) == planes.numel()
            glowmi.conv2d_pack_filter(G.dev(np.ascontiguousarray(w.T)), desc, planes)
        glowmi.fc_packed(ad, wd, planes, bd, y, M, K, N, wl.ACT_RELU, G.workspace(glowmi.fc_packed_workspace_bytes(M, K, N)))
    torch.cuda.synchronize()
    variant = glowmi.last_variant()
    assert variant.startswith("igemm_f32_p3_fc"), variant
    assert variant.endswith("_longk") == ((-(-K // 64) + max(split, 1) - 1) // max(split, 1) > 16), variant
    assert G.guards_intact(whole, torch.float32), "write outside the output"
    scale = np.where(np.arange(M) % 3 == 0, np.float32(2.0 ** 20), np.float32(1.0))[:, None]   # a row's results scale with it
    G.assert_close_f32(y.cpu().numpy() / scale, ref / scale, f"fc over planes {case} {order}")


@pytest.mark.parametrize("M,K,N", [(1152, 9216, 128), (1152, 4608, 256)])
def test_sums_folded_in_turn_lie_no_farther_from_64_bit_ones(M, K, N, knobs):
    """Long reductions fold the sums of a workgroup's two halves into one set of totals.  The same product as a pointwise convolution over the
    same planes (igemm_f32_p3: as many products to a chain, totals of each half's own) says how far sums of this kind lie from 64-bit ones; a
    hundredth is what the order alone changes."""
    import gpu_util as G
    import torch
    import paper_1805_00907_amd as glowmi
    for name, value in (("F32_P3_MIN_M", 1), ("F32_P3_RATIO", 0), ("F32_SPLIT", 1)):
        knobs.set(name, value)
    rng = np.random.default_rng(47500 + K)
    a = rng.standard_normal((M, K)).astype(np.float32)
    w = (rng.standard_normal((K, N)) / np.sqrt(K)).astype(np.float32)
    exact = a.astype(np.float64) @ w.astype(np.float64)
    ad, wd, y = G.dev(a), G.dev(w), G.poison((M, N), torch.float32)
    planes = torch.empty(glowmi.fc_filter_planes_bytes(K, N), dtype=torch.uint8, device="cuda:0")
    glowmi.fc_pack_filter(wd, K, N, planes)
    glowmi.fc_packed(ad, wd, planes, None, y, M, K, N, wl.ACT_NONE, G.workspace(glowmi.fc_packed_workspace_bytes(M, K, N)))
    torch.cuda.synchronize()
    assert glowmi.last_variant() == "igemm_f32_p3_fc_128x128_longk"
    got = np.linalg.norm(y.cpu().numpy() - exact)
    knobs.set("F32_PATCH", 0)
    desc = glowmi.ConvDesc(1, M, 1, K, N, 1, 1, 1, 1, 0, 0, 0, 0, 1)
    z = G.poison((1, M, 1, N), torch.float32)
    glowmi.conv2d(ad, G.dev(np.ascontiguousarray(w.T)), None, z, desc, wl.ACT_NONE, G.workspace(glowmi.conv2d_workspace_bytes(desc)))
    torch.cuda.synchronize()
    assert glowmi.last_variant().startswith("igemm_f32_p3_128x128") and glowmi.last_variant().endswith("longk"), glowmi.last_variant()
    reference = np.linalg.norm(z.cpu().numpy().reshape(M, N) - exact)
    print(f"distances {got / np.linalg.norm(exact):.3e} and {reference / np.linalg.norm(exact):.3e}")
    assert got <= 1.01 * reference, (got, reference)
