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
