"""fp32 FullyConnected with one to four rows in one launch (fc_rows_f32) against the CPU oracle: reductions shorter than a
pass, of whole passes and ragged, columns that end inside a lane's four, and which layers take it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 500, 130), (2, 64, 7), (3, 1537, 777), (4, 1024, 64), (1, 2048, 1000), (4, 8192, 33),
                                   (2, 513, 65), (1, 8191, 5)], ids=lambda s: "x".join(map(str, s)))
def test_fc_rows_f32(shape, knobs):
    import gpu_util as G
    m, k, n = shape
    knobs.set("F32_FC_ROWS", 2)
    rng = np.random.default_rng(38000 + m + k + n)
    a = rng.uniform(-1, 1, size=(m, k)).astype(np.float32)
    w = (rng.uniform(-1, 1, size=(k, n)) / np.sqrt(k)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(n,)).astype(np.float32)
    for bias, act in ((b, wl.ACT_RELU), (None, wl.ACT_NONE)):
        got, variant = G.gpu_fc_f32(a, w, bias, act)
        assert variant == "fc_rows_f32", variant
        G.assert_close_f32(got, oracle.fc_f32(a, w, bias, act=act), f"{shape} [{variant}]")


@pytest.mark.parametrize("shape,taken", [((1, 512, 1000), True), ((1, 4096, 4096), False), ((4, 2048, 1000), False), ((4, 1024, 77), True),
                                         ((5, 1024, 77), False)], ids=str)
def test_fc_rows_f32_choice(shape, taken):
    import gpu_util as G
    m, k, n = shape
    rng = np.random.default_rng(38100 + m + k + n)
    a, w = rng.standard_normal((m, k), dtype=np.float32), rng.standard_normal((k, n), dtype=np.float32)
    _, variant = G.gpu_fc_f32(a, w, None, wl.ACT_NONE)
    assert (variant == "fc_rows_f32") == taken, variant
