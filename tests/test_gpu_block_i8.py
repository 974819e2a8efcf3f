"""1x1, 3x3, 1x1 of an int8 sequence in one launch (block_i8.hip) against the oracle's chain, code for code: channel counts that fill
no chunk, tap or block of channels, maps smaller than a tile and ones that cut it, several tiles to a workgroup, and what stays three launches; runs
anywhere in a longer sequence."""
import numpy as np
import pytest

import oracle
from paper_1805_00907_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _gpu():
    import gpu_util
    return gpu_util


class Block:
    def __init__(self, n, h, w, c, mid, k, add, seed, act=True, w_off=0):
        import paper_1805_00907_amd as glowmi
        G = _gpu()
        shapes = [(c, mid, 1), (mid, mid, 3), (mid, k, 1)]
        specs = [wl.ConvLayer(f"b{i}", n, h, w, ci, co, r, r, 1, r // 2, act=act, add=add and i == 2) for i, (ci, co, r) in enumerate(shapes)]
        data = [wl.conv_inputs_q(s, seed + i, w_off=w_off) for i, s in enumerate(specs)]
        qps = [d[3] for d in data]
        in_q = [(qps[0].x_scale, qps[0].x_off)] + [(q.y_scale, q.y_off) for q in qps[:2]]
        self.x, self.shape, self.keep = data[0][0], (n, h, w, k), []
        self.xq = glowmi.QParam(*in_q[0])
        self.tuples, ref = [], self.x
        for i, s in enumerate(specs):
            _, wt, b, qp = data[i]
            b = None if i == 1 and seed % 2 else b                    # a layer without a bias
            wd, bd = G.dev(wt), None if b is None else G.dev(b)
            self.keep += [wd, bd]
            self.tuples.append((G.desc_of(s), wd, bd, s.act, s.add, glowmi.QParam(qp.w_scale, qp.w_off), glowmi.QParam(qp.y_scale, qp.y_off)))
            ref = oracle.qconv2d_add(ref, in_q[i][0], in_q[i][1], wt, qp.w_scale, qp.w_off, b, self.x if s.add else None, in_q[0][0],
                                     in_q[0][1], qp.y_scale, qp.y_off, (1, 1), (s.pad,) * 4, 1, act=s.act)
        self.ref = ref

    def run(self, x=None, y=None, stream=None):
        import torch
        import paper_1805_00907_amd as glowmi
        G = _gpu()
        arr = glowmi.seq_layers(self.tuples)
        arena = torch.empty(glowmi.seq_arena_bytes(arr, True), dtype=torch.uint8, device="cuda:0")
        xd = G.dev(self.x) if x is None else x
        whole, out = G.guarded(self.shape, torch.int8) if y is None else (None, y)
        glowmi.seq_qconv2d(xd, self.xq, arr, out, arena)
        torch.cuda.synchronize()
        if whole is not None:
            assert G.guards_intact(whole, torch.int8), "write outside the output tensor"
        return out.cpu().numpy(), glowmi.last_variant()


@pytest.mark.parametrize("n,h,w,c,mid,k,add", [
    (1, 1, 1, 32, 4, 16, False), (1, 7, 7, 128, 32, 128, True), (2, 5, 9, 96, 28, 96, True), (3, 2, 3, 64, 20, 48, False),
    (1, 9, 13, 160, 40, 160, True), (2, 11, 6, 256, 64, 256, True), (1, 14, 30, 224, 56, 224, True), (2, 6, 7, 32, 36, 256, False),
    (1, 10, 10, 384, 96, 384, True), (2, 7, 12, 288, 72, 288, True), (1, 8, 5, 320, 84, 16, False), (1, 3, 40, 352, 88, 352, True),
])
@pytest.mark.parametrize("act", [True, False])
def test_every_code_of_a_block_is_the_oracles(n, h, w, c, mid, k, add, act, knobs):
    knobs.set("I8_BLOCK", 2)
    b = Block(n, h, w, c, mid, k, add, 9100 + mid + h, act)
    got, variant = b.run()
    assert variant.startswith("block_i8"), variant
    _gpu().assert_equal_i8(got, b.ref, variant)


@pytest.mark.parametrize("n,h,w,c,mid,th,tw", [(9, 33, 35, 128, 32, 2, 3), (5, 29, 31, 256, 64, 3, 2), (6, 20, 31, 288, 72, 2, 4),
                                                (2, 40, 44, 256, 64, 14, 14), (2, 15, 15, 256, 64, 15, 13), (1, 2, 62, 128, 32, 2, 62)])
def test_several_tiles_to_a_workgroup_and_large_tiles(n, h, w, c, mid, th, tw, knobs):
    knobs.set("I8_BLOCK", 2)
    b = Block(n, h, w, c, mid, c, True, 9300 + mid)
    for forced in (True, False):
        if forced:
            knobs.set("I8_BLOCK_TH", th)
            knobs.set("I8_BLOCK_TW", tw)
        else:
            knobs.set("I8_BLOCK_TH", 0)
            knobs.set("I8_BLOCK_TW", 0)
        got, variant = b.run()
        assert variant.startswith("block_i8"), variant
        _gpu().assert_equal_i8(got, b.ref, variant)


def test_graph_replays_give_what_the_eager_call_gives(knobs):
    import torch
    import paper_1805_00907_amd as glowmi
    G = _gpu()
    b = Block(2, 14, 14, 256, 64, 256, True, 9401)
    arr = glowmi.seq_layers(b.tuples)
    arena = torch.empty(glowmi.seq_arena_bytes(arr, True), dtype=torch.uint8, device="cuda:0")
    xd, y = G.dev(b.x), G.poison(b.shape, torch.int8)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        glowmi.seq_qconv2d(xd, b.xq, arr, y, arena, side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            glowmi.seq_qconv2d(xd, b.xq, arr, y, arena, side)
    assert glowmi.last_variant().startswith("block_i8")
    for _ in range(3):
        y.fill_(99)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        G.assert_equal_i8(y.cpu().numpy(), b.ref, "graph replay")
        float(torch.empty(1 << 16, device="cuda:0").normal_().sum())


# layers as (output channels, filter size), which of them add the sequence's input, x's channels
LONGER = {
    "block, layer": ([(32, 1), (32, 3), (128, 1), (128, 3)], (2, 3), 128),
    "layer, block": ([(128, 3), (32, 1), (32, 3), (128, 1)], (3,), 128),
    "layer, block, layer": ([(96, 1), (28, 1), (28, 3), (112, 1), (64, 1)], (), 64),
    "block, block": ([(64, 1), (64, 3), (256, 1), (56, 1), (56, 3), (256, 1)], (2, 5), 256),
    "layer, block, block": ([(128, 1), (32, 1), (32, 3), (128, 1), (24, 1), (24, 3), (96, 1)], (6,), 96),
}


@pytest.mark.parametrize("layers,add,c", LONGER.values(), ids=LONGER)
@pytest.mark.parametrize("in_place", [False, True], ids=["", "over_its_input"])
@pytest.mark.parametrize("mode", [2, 0], ids=["blocks", "layers"])
def test_longer_sequences(layers, add, c, in_place, mode, knobs):
    """Runs that begin behind a layer (their input is a region of the arena, the addend the sequence's x), stand in front of one or of each
    other, and write over x, which the last one's addend still is."""
    import torch
    import paper_1805_00907_amd as glowmi
    G = _gpu()
    knobs.set("I8_BLOCK", mode)
    n, h, w = 2, 9, 11
    specs, ci = [], c
    for i, (k, r) in enumerate(layers):
        specs.append(wl.ConvLayer(f"s{i}", n, h, w, ci, k, r, r, 1, r // 2, act=True, add=i in add))
        ci = k
    data = [wl.conv_inputs_q(s, 9700 + 10 * len(layers) + i) for i, s in enumerate(specs)]
    qps = [d[3] for d in data]
    in_q = [(qps[0].x_scale, qps[0].x_off)] + [(q.y_scale, q.y_off) for q in qps[:-1]]
    x = ref = data[0][0]
    tuples, keep = [], []
    for i, s in enumerate(specs):
        _, wt, b, qp = data[i]
        wd, bd = G.dev(wt), G.dev(b)
        keep += [wd, bd]
        tuples.append((G.desc_of(s), wd, bd, s.act, s.add, glowmi.QParam(qp.w_scale, qp.w_off), glowmi.QParam(qp.y_scale, qp.y_off)))
        ref = oracle.qconv2d_add(ref, in_q[i][0], in_q[i][1], wt, qp.w_scale, qp.w_off, b, x if s.add else None, in_q[0][0], in_q[0][1],
                                 qp.y_scale, qp.y_off, (1, 1), (s.pad,) * 4, 1, act=s.act)
    arr = glowmi.seq_layers(tuples)
    arena, arena_guard = torch.full((glowmi.seq_arena_bytes(arr, True) + 4096,), 0x5a, dtype=torch.uint8, device="cuda:0"), 4096
    xd = G.dev(x)
    whole, y = (None, xd) if in_place else G.guarded((n, h, w, layers[-1][0]), torch.int8)
    glowmi.seq_qconv2d(xd, glowmi.QParam(*in_q[0]), arr, y, arena[:-arena_guard])
    torch.cuda.synchronize()
    variant = glowmi.last_variant()
    if layers[-2][1] == 3:                                    # a run is the last launch
        assert variant.startswith("block_i8") == (mode == 2), variant
    assert whole is None or G.guards_intact(whole, torch.int8), "write outside the output tensor"
    assert bool((arena[-arena_guard:] == 0x5a).all()), "write behind the arena"
    G.assert_equal_i8(y.cpu().numpy(), ref, variant)
    assert 0.02 < np.mean((ref > -128) & (ref < 127)), "almost everything saturates"


def test_what_stays_three_launches(knobs):
    """An output over the input (neighbouring tiles read it after this one's output is written), filters with an offset in their
    codes, the switch."""
    import torch
    G = _gpu()
    b = Block(2, 9, 9, 128, 32, 128, True, 9500)
    xd = G.dev(b.x)
    got, variant = b.run(x=xd, y=xd)
    assert not variant.startswith("block_i8"), variant
    G.assert_equal_i8(got, b.ref, "in place")
    offset = Block(1, 9, 9, 128, 32, 128, True, 9510, w_off=3)
    got, variant = offset.run()
    assert not variant.startswith("block_i8"), variant
    G.assert_equal_i8(got, offset.ref, "filters with an offset")
    knobs.set("I8_BLOCK", 0)
    got, variant = b.run()
    assert not variant.startswith("block_i8"), variant
    G.assert_equal_i8(got, b.ref, "switched off")
