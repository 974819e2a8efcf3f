"""3x3 layers whose reduction conv_patch_f32 takes in parts: every form and number of parts on ragged maps and channels against the CPU
oracle, with the add link and in place; what the planner gives it, and that a workspace without room for the parts runs what ran
without them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


def _gpu():
    import gpu_util
    return gpu_util


# n  h  w  c  k  stride
SHAPES = [
    (1, 9, 9, 72, 40, 1),                # a last chunk of eight channels
    (2, 7, 13, 200, 72, 1),
    (3, 5, 6, 97, 33, 1),                # channels by value
    (1, 15, 17, 136, 130, 2),
    (2, 8, 8, 320, 128, 2),
]


@pytest.mark.parametrize("parts", [2, 3, 8])
@pytest.mark.parametrize("shape,form", [(s, f) for s in SHAPES for f in range(6) if s[5] == 1 or f == 1],     # (stride 2 has one form)
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_parts(shape, form, parts, knobs):
    G = _gpu()
    n, h, w, c, k, st = shape
    chunk = (64, 32, 128, 32, 32, 32)[form]
    chunks = (c + chunk - 1) // chunk
    each = (chunks + parts - 1) // parts
    whole = (chunks + each - 1) // each != parts        # no such number of parts: not a launch
    for name, value in (("F32_PATCH", 2), ("F32_SHORT", 0), ("F32_FEW", 0), ("F32_PATCH_TILE", form), ("F32_PATCH_PARTS", parts)):
        knobs.set(name, value)
    rng = np.random.default_rng(93000 + c + k + form)
    x = rng.uniform(-1, 1, size=(n, h, w, c)).astype(np.float32)
    wt = (rng.uniform(-1, 1, size=(k, 3, 3, c)) / np.sqrt(9 * c)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, size=(k,)).astype(np.float32)
    desc = G.make_desc(x.shape, wt.shape, (st, st), (1, 1, 1, 1), 1)
    ref = oracle.conv2d_f32(x, wt, b, (st, st), (1, 1, 1, 1), 1, act=wl.ACT_RELU)
    got, variant = G.gpu_conv2d_f32(x, wt, b, desc, wl.ACT_RELU, use_workspace=True)
    assert variant.endswith("_parts") != whole, variant
    G.assert_close_f32(got, ref, f"{shape} [{variant}]")
    add = rng.uniform(-1, 1, size=ref.shape).astype(np.float32)
    ref = oracle.conv2d_f32_add(x, wt, b, add, (st, st), (1, 1, 1, 1), 1, act=wl.ACT_RELU)
    for in_place in (False, True):
        got, variant = G.gpu_conv2d_f32_chain(x, wt, b, add, desc, wl.ACT_RELU, in_place=in_place)
        assert variant.endswith("_parts") != whole, variant
        G.assert_close_f32(got, ref, f"{shape} add [{variant}]")


@pytest.mark.parametrize("n,h,c,k,stride,parts", [(16, 14, 512, 512, 2, True), (32, 14, 512, 512, 2, True), (16, 56, 128, 128, 2, False), (8, 28, 128, 128, 1, False)])
def test_planned(n, h, c, k, stride, parts, knobs):
    import torch
    import paper_1805_00907_amd as glowmi
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    x = torch.randn((n, h, h, c), generator=gen, device="cuda:0")
    w = torch.randn((k, 3, 3, c), generator=gen, device="cuda:0") / (9 * c) ** 0.5
    b = torch.randn((k,), generator=gen, device="cuda:0")
    desc = glowmi.ConvDesc(n, h, h, c, k, 3, 3, stride, stride, 1, 1, 1, 1, 1)
    oh = (h - 1) // stride + 1
    outs, names = [], []

    def call(nbytes):
        y = torch.full((n, oh, oh, k), float("nan"), device="cuda:0")
        glowmi.conv2d(x, w, b, y, desc, glowmi.ACT_RELU, torch.empty(nbytes, dtype=torch.uint8, device="cuda:0"))
        outs.append(y.double())
        names.append(glowmi.last_variant())

    call(glowmi.conv2d_workspace_bytes(desc))
    knobs.set("F32_PATCH_PARTS", 1)
    call(glowmi.conv2d_workspace_bytes(desc))
    glowmi.tuning_reset()
    call((9 * c * k + k) * 4 + 4096)                    # room for the filter's planes alone
    assert [name.endswith("_parts") for name in names] == [parts, False, False], names
    # ways to sum 4608 products of unit variance in short runs of 32 bits: each within some 2e-7 of the sums' norm
    for other in outs[1:]:
        assert float((outs[0] - other).norm() / outs[0].norm()) < 1e-6, names


def test_layers_of_a_sequence_run_whole(knobs):
    """A layer that runs in parts by itself, and next to one that wants more scratch than its parts: in a sequence it is what the same calls
    without parts give, bit for bit."""
    import torch
    import paper_1805_00907_amd as glowmi
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(9)
    x = torch.randn((16, 5, 7, 840), generator=gen, device="cuda:0")
    descs = [glowmi.ConvDesc(16, 5, 7, c, k, 3, 3, 1, 1, 1, 1, 1, 1, 1) for c, k in ((840, 248), (248, 1024))]
    ws = [torch.randn((d.k, 3, 3, d.c), generator=gen, device="cuda:0") / (9 * d.c) ** 0.5 for d in descs]
    bs = [torch.randn((d.k,), generator=gen, device="cuda:0") for d in descs]

    def one_by_one():
        at, names = x, []
        for d, w, b in zip(descs, ws, bs):
            y = torch.full((16, 5, 7, d.k), float("nan"), device="cuda:0")
            nbytes = glowmi.conv2d_workspace_bytes(d)
            glowmi.conv2d(at, w, b, y, d, glowmi.ACT_RELU, torch.empty(nbytes, dtype=torch.uint8, device="cuda:0") if nbytes else None)
            names.append(glowmi.last_variant())
            at = y
        return at, names

    assert one_by_one()[1][0].endswith("_parts")
    layers = glowmi.seq_layers([(d, w, b, glowmi.ACT_RELU, False) for d, w, b in zip(descs, ws, bs)])
    y = torch.full((16, 5, 7, 1024), float("nan"), device="cuda:0")
    glowmi.seq_conv2d(x, layers, y, torch.empty(glowmi.seq_arena_bytes(layers, False), dtype=torch.uint8, device="cuda:0"))
    knobs.set("F32_PATCH_PARTS", 1)
    want, names = one_by_one()
    torch.cuda.synchronize()
    assert not names[0].endswith("_parts") and torch.equal(y, want), names
