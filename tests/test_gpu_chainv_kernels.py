"""Op lists that fold into the clamp of a kernel's epilogue (at most one tensor add, then bounds; int8: multiplies anywhere), on
every kernel that they reach, against the oracle element by element: bounds on both sides, several in a row, bounds that
coincide or lie outside what the output can hold, behind an added tensor, in place.  fp32: |gpu - oracle| <= 1e-5 + 1e-4
|oracle|; int8: bit for bit.  And on NaN and infinities the folded clamp gives what the ops in turn give."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1805_00907_amd import workloads as wl


def _gpu():
    import gpu_util
    return gpu_util


NO_K3 = {"F32_K3": 0, "F32_K3C64": 0}
P3 = {"F32_P3_MIN_M": 1, "F32_P3_RATIO": 0, "F32_PATCH": 0, **NO_K3}

# name: knobs, (n, h, w, c, k, r, stride, pad, groups), kernel without an added tensor, the same kernel takes one
F32 = {
    "dw_s1": ({}, (2, 9, 11, 22, 22, 3, 1, 1, 22), "conv_dw_f32_3x3s1", False),
    "dw_s2": ({}, (2, 12, 11, 24, 24, 3, 2, 1, 24), "conv_dw_f32_3x3s2", False),
    "first_fp32": ({"F32_SMALLC_BF16": 0}, (1, 30, 26, 3, 40, 7, 2, 3, 1), "conv_smallc_f32", False),
    "first_f16": ({"F32_SMALLC_BF16": 1}, (1, 30, 26, 3, 72, 7, 2, 3, 1), "conv_smallc_f32", False),
    "first_3x3": ({}, (1, 17, 26, 3, 40, 3, 1, 1, 1), "conv_smallc_f32", False),
    "first_3x3s2": ({}, (1, 17, 26, 3, 72, 3, 2, 1, 1), "conv_smallc_f32", False),
    "pw64": ({"F32_PW_MIN_ITEMS": 1, "F32_PW_BF16": 0}, (2, 9, 9, 64, 70, 1, 1, 0, 1), "conv_pw_f32", True),
    "pw128": ({"F32_PW_MIN_ITEMS": 1, "F32_PW_BF16": 0}, (2, 9, 9, 128, 64, 1, 2, 0, 1), "conv_pw_f32", True),
    "pw256": ({"F32_PW_MIN_ITEMS": 1, "F32_PW_BF16": 0}, (1, 9, 9, 256, 64, 1, 1, 0, 1), "conv_pw_f32", True),
    "pw64_bf16": ({"F32_PW_MIN_ITEMS": 1, "F32_PW_BF16": 1}, (2, 9, 9, 64, 70, 1, 1, 0, 1), "conv_pw_f32", True),
    "pw256_bf16": ({"F32_PW_MIN_ITEMS": 1, "F32_PW_BF16": 1}, (1, 9, 9, 256, 64, 1, 1, 0, 1), "conv_pw_f32", True),
    "k3c64": ({"F32_K3C64_MIN_TILES": 1}, (2, 19, 21, 64, 72, 3, 1, 1, 1), "conv_k3c64_f32", True),
    "k3_fixed": ({"F32_K3_ANY": 1, "F32_K3C64": 0, "F32_K3V": 0}, (1, 19, 21, 96, 136, 3, 1, 1, 1), "conv_k3_f32", True),
    "k3_wide": ({"F32_K3_ANY": 1, "F32_K3C64": 0, "F32_K3V": 0}, (1, 19, 21, 96, 40, 3, 1, 1, 1), "conv_k3_f32", True),
    "k3_shaped": ({"F32_K3_ANY": 1, "F32_K3C64": 0, "F32_K3V": 1}, (1, 19, 21, 96, 136, 3, 1, 1, 1), "conv_k3_f32", True),
    "p3_128": ({**P3, "F32_P3_BN": 128, "F32_SPLIT": 1}, (1, 14, 13, 72, 136, 3, 1, 1, 1), "igemm_f32_p3_128x128", True),
    "p3_64": ({**P3, "F32_P3_BN": 64, "F32_SPLIT": 1}, (1, 14, 13, 72, 72, 3, 2, 1, 1), "igemm_f32_p3_128x64", True),
    "p3_split": ({**P3, "F32_SPLIT": 3}, (1, 14, 13, 72, 136, 3, 1, 1, 1), "igemm_f32_p3", True),
    "patch_3x3": ({"F32_PATCH": 2, **NO_K3}, (2, 9, 13, 40, 24, 3, 1, 1, 1), "conv_patch_f32", True),
    "patch_3x3s2": ({"F32_PATCH": 2, **NO_K3}, (2, 9, 13, 40, 24, 3, 2, 1, 1), "conv_patch_f32", True),
    "patch_1x1": ({"F32_PATCH": 2}, (2, 11, 9, 72, 100, 1, 1, 0, 1), "conv_patch_f32", True),
    "small": ({"F32_PATCH": 0, "F32_FEW": 0}, (1, 7, 7, 48, 48, 3, 1, 1, 1), "conv_small_f32", False),
    "few0": ({"F32_FEW": 2, "F32_FEW_TILE": 0}, (1, 7, 7, 48, 50, 3, 1, 1, 1), "conv_few_f32_16x16w4", True),
    "few1": ({"F32_FEW": 2, "F32_FEW_TILE": 1}, (1, 9, 8, 64, 36, 3, 2, 1, 1), "conv_few_f32_16x16w8", True),
    "few2": ({"F32_FEW": 2, "F32_FEW_TILE": 2}, (2, 7, 8, 21, 40, 3, 1, 1, 1), "conv_few_f32_16x32w4", True),
    "short1": ({"F32_SHORT": 2, "F32_SHORT_FORM": 1}, (2, 9, 13, 72, 50, 1, 1, 0, 1), "conv_short_f32_32x32", True),
    "short2": ({"F32_SHORT": 2, "F32_SHORT_FORM": 2}, (2, 9, 13, 96, 70, 1, 2, 0, 1), "conv_short_f32_32x64", True),
    "short4": ({"F32_SHORT": 2, "F32_SHORT_FORM": 4}, (1, 11, 13, 20, 130, 1, 1, 0, 1), "conv_short_f32_32x128", True),
    "small_split": ({"F32_PATCH": 0, "F32_SMALL_MIN_WGS": 1}, (1, 7, 7, 512, 96, 3, 1, 1, 1), "conv_small_f32", True),
    "tile0_long": ({"F32_TILE": 0, "F32_SPLIT": 1}, (1, 6, 6, 2080, 33, 1, 1, 0, 1), "igemm_f32_64x64w4", True),
    "tile0_split": ({"F32_TILE": 0, "F32_SPLIT": 4}, (1, 6, 6, 480, 33, 3, 1, 1, 1), "igemm_f32_64x64w4", True),
    "tile1": ({"F32_TILE": 1}, (1, 15, 15, 20, 72, 3, 1, 1, 1), "igemm_f32_128x64w8", True),
    "tile2": ({"F32_TILE": 2}, (1, 15, 15, 20, 72, 3, 1, 1, 2), "igemm_f32_128x128w8", True),
    "tile3": ({"F32_TILE": 3}, (1, 15, 15, 21, 72, 3, 1, 1, 1), "igemm_f32_32x128w4", True),
    "tile5": ({"F32_TILE": 5}, (1, 15, 15, 20, 140, 3, 1, 1, 1), "igemm_f32_128x128w4", True),
}


def _lists_f32(t):
    return [
        [("clip", -0.25, 0.4)],
        [("max", 0.125)],
        [("max", -0.3), ("clip", -0.5, 0.2), ("max", -0.1)],
        [("clip", 0.1, 0.1)],
        [("clip", -np.inf, 0.3)],
        [("clip", 5.0, 6.0)],
        [("add", t), ("clip", -0.3, 0.5)],
        [("add", t), ("max", -0.2), ("clip", -1.0, 0.75)],
    ]


def _f32_inputs(seed, n, h, w, c, k, r, g):
    rng = np.random.default_rng(seed)
    x = rng.uniform(-1, 1, size=(n, h, w, c)).astype(np.float32)
    wt = (rng.standard_normal(size=(k, r, r, c // g)) / np.sqrt(r * r * c // g)).astype(np.float32)
    return x, wt, rng.uniform(-0.1, 0.1, size=(k,)).astype(np.float32), rng


@pytest.mark.parametrize("name", F32)
def test_folded_lists_f32(name, knobs):
    import torch
    import paper_1805_00907_amd as glowmi
    G = _gpu()
    settings, (n, h, w, c, k, r, st, pd, g), kernel, adds = F32[name]
    for knob, value in settings.items():
        knobs.set(knob, value)
    x, wt, b, rng = _f32_inputs(41000 + c + k, n, h, w, c, k, r, g)
    desc = G.make_desc(x.shape, wt.shape, (st, st), (pd,) * 4, g)
    yshape = (n, *glowmi.conv_out_shape(desc), k)
    t = rng.uniform(-1, 1, size=yshape).astype(np.float32)
    xd, wd, bd, td = G.dev(x), G.dev(wt), G.dev(b), G.dev(t)
    for ops in _lists_f32(t):
        ref = oracle.conv2d_f32_chain(x, wt, b, ops, (st, st), (pd,) * 4, g)
        added = ops[0][0] == "add"
        for in_place in (False, True) if added else (False,):
            whole, y = G.guarded(yshape, torch.float32)
            if in_place:
                y.copy_(td)
            dev_ops = [("add", y if in_place else td) if o[0] == "add" else o for o in ops]
            ws = G.workspace(glowmi.conv2d_chainv_workspace_bytes(desc, dev_ops))
            glowmi.conv2d_chainv(xd, wd, bd, y, desc, dev_ops, ws)
            torch.cuda.synchronize()
            variant = glowmi.last_variant()
            what = f"{name} {[o[:1] + o[1:] if o[0] != 'add' else o[0] for o in ops]} in place {in_place} [{variant}]"
            assert G.guards_intact(whole, torch.float32), what
            assert variant.endswith("_chainv") and (variant.startswith(kernel) or (added and not adds)), what
            G.assert_close_f32(y.cpu().numpy(), ref, what)


@pytest.mark.parametrize("name", ["dw_s1", "first_fp32", "pw64", "small", "few0", "few2", "tile1"])
def test_folded_clamp_takes_nan_and_infinities_as_the_ops_in_turn(name, knobs):
    """On kernels that multiply in fp32: a NaN becomes the lower bound (the result of max, then min), an infinity the bound
    on its side, as where the ops run one by one."""
    import torch
    import paper_1805_00907_amd as glowmi
    G = _gpu()
    settings, (n, h, w, c, k, r, st, pd, g), kernel, _ = F32[name]
    x, wt, b, rng = _f32_inputs(41500, n, h, w, c, k, r, g)
    for i, v in enumerate((np.nan, np.inf, -np.inf)):
        x[0, 3 + i, 2 + 2 * i, (5 * i) % c] = v
    desc = G.make_desc(x.shape, wt.shape, (st, st), (pd,) * 4, g)
    yshape = (n, *glowmi.conv_out_shape(desc), k)
    xd, wd, bd = G.dev(x), G.dev(wt), G.dev(b)
    for ops in ([("max", 0.0)], [("clip", -0.25, 0.4)], [("max", -0.1)]):
        out = []
        for alone in (False, True):
            for knob, value in settings.items():
                knobs.set(knob, value)
            y = G.poison(yshape, torch.float32)
            given = ops + [("mul", 1.0)] if alone else ops      # a multiply last keeps the list from folding
            glowmi.conv2d_chainv(xd, wd, bd, y, desc, given, G.workspace(glowmi.conv2d_chainv_workspace_bytes(desc, given)))
            torch.cuda.synchronize()
            assert alone or glowmi.last_variant().startswith(kernel), glowmi.last_variant()
            out.append(y.cpu().numpy())
        G.assert_close_f32(np.nan_to_num(out[0], posinf=1e30), np.nan_to_num(out[1], posinf=1e30), f"{name} {ops}")


I8 = {
    "dw_s1": ({}, (2, 9, 11, 22, 22, 3, 1, 1, 22), 0, "conv_dw_i8", False),
    "dw_s1_off": ({}, (2, 9, 11, 24, 24, 3, 1, 1, 24), -7, "conv_dw_i8", False),
    "dw_s2": ({}, (2, 12, 11, 24, 24, 3, 2, 1, 24), 0, "conv_dw_i8", False),
    "first": ({}, (1, 30, 26, 3, 40, 7, 2, 3, 1), 0, "conv_smallc_i8", False),
    "first_3x3": ({}, (1, 17, 26, 3, 72, 3, 1, 1, 1), 0, "conv_smallc_i8", False),
    "pw64": ({"I8_PW_MIN_ITEMS": 1}, (2, 9, 9, 64, 80, 1, 1, 0, 1), 0, "conv_pw_i8", True),
    "pw128": ({"I8_PW_MIN_ITEMS": 1}, (2, 9, 9, 128, 64, 1, 2, 0, 1), 0, "conv_pw_i8", True),
    "pw256": ({"I8_PW_MIN_ITEMS": 1}, (1, 9, 9, 256, 64, 1, 1, 0, 1), 0, "conv_pw_i8", True),
    "k3c64_w8": ({"I8_K3_MIN_BLOCKS": 1, "I8_K3_WAVES": 8}, (1, 19, 21, 64, 80, 3, 1, 1, 1), 0, "conv_k3c64_i8_w8", True),
    "k3c64_w16": ({"I8_K3_MIN_BLOCKS": 1, "I8_K3_WAVES": 16}, (1, 19, 21, 64, 80, 3, 1, 1, 1), 0, "conv_k3c64_i8_w16", True),
    "k3c64_gather": ({"I8_K3_MIN_BLOCKS": 1, "I8_K3_GATHER": 1}, (1, 19, 21, 64, 80, 3, 2, 1, 1), 0, "conv_k3c64_i8", True),
    "wide128": ({"I8_TILE": 4}, (1, 15, 15, 80, 140, 3, 1, 1, 1), 0, "igemm_i8_wide", True),
    "wide64": ({"I8_TILE": 5}, (1, 15, 15, 80, 140, 3, 1, 1, 1), 3, "igemm_i8_wide", True),
    "wide_split": ({"I8_TILE": 4, "I8_WIDE_SPLIT": 3}, (1, 15, 15, 160, 140, 3, 1, 1, 1), 0, "igemm_i8_wide", True),
    "small": ({"I8_SMALL_MAX_TILES": 100000}, (1, 13, 9, 40, 50, 3, 1, 1, 1), -5, "conv_small_i8", True),
    "small_split": ({"I8_FEW": 0}, (1, 7, 7, 512, 96, 3, 1, 1, 1), 0, "conv_small_i8", True),
    "few0": ({"I8_FEW": 2, "I8_FEW_TILE": 0}, (1, 7, 7, 128, 50, 3, 1, 1, 1), 0, "conv_few_i8_16x16w4", True),
    "few1": ({"I8_FEW": 2, "I8_FEW_TILE": 1}, (1, 9, 8, 100, 36, 3, 2, 1, 1), 5, "conv_few_i8_16x16w8", True),
    "few2": ({"I8_FEW": 2, "I8_FEW_TILE": 2}, (2, 7, 5, 21, 40, 3, 1, 1, 1), 0, "conv_few_i8_16x32w4", True),
    "short1": ({"I8_SHORT": 2, "I8_SHORT_FORM": 1}, (2, 9, 13, 72, 52, 3, 1, 1, 1), 0, "conv_short_i8_32x32", True),
    "short2": ({"I8_SHORT": 2, "I8_SHORT_FORM": 2}, (2, 9, 13, 128, 72, 1, 2, 0, 1), 0, "conv_short_i8_32x64", True),
    "short_odd": ({"I8_SHORT": 2, "I8_SHORT_FORM": 2}, (2, 9, 13, 23, 70, 1, 1, 0, 1), 0, "conv_short_i8_32x64", False),
    "tile0": ({"I8_TILE": 0}, (1, 13, 9, 40, 50, 3, 1, 1, 1), 4, "igemm_i8_64x64w4", True),
    "tile0_split": ({"I8_TILE": 0, "I8_SPLIT": 3}, (1, 6, 6, 480, 33, 3, 1, 1, 1), 0, "igemm_i8_64x64w4", True),
    "tile1": ({"I8_TILE": 1}, (1, 13, 13, 40, 70, 3, 1, 1, 1), 0, "igemm_i8_128x64w8", True),
    "tile2": ({"I8_TILE": 2}, (1, 13, 13, 40, 140, 3, 1, 1, 1), 0, "igemm_i8_128x128w8", True),
    "tile6": ({"I8_TILE": 6}, (1, 13, 13, 40, 70, 3, 1, 1, 2), 0, "igemm_i8_64x64w4k2", True),
    "tile7": ({"I8_TILE": 7}, (1, 13, 13, 40, 70, 3, 1, 1, 1), 0, "igemm_i8_64x64w4k4", True),
}


@pytest.mark.parametrize("name", I8)
def test_folded_lists_i8(name, knobs):
    import torch
    import paper_1805_00907_amd as glowmi
    G = _gpu()
    settings, (n, h, w, c, k, r, st, pd, g), w_off, kernel, adds = I8[name]
    for knob, value in settings.items():
        knobs.set(knob, value)
    xq, wq, bq, qp = wl.conv_inputs_q(wl.ConvLayer("fold", n, h, w, c, k, r, r, st, pd, g), 42000 + c + k, dist="normal",
                                      w_off=w_off)
    desc = G.make_desc(xq.shape, wq.shape, (st, st), (pd,) * 4, g)
    yshape = (n, *glowmi.conv_out_shape(desc), k)
    rng = np.random.default_rng(42500)
    t = rng.integers(-128, 128, size=yshape, dtype=np.int8)
    tq = (float(np.float32(qp.y_scale * 0.7)), 9)
    sy = qp.y_scale
    lo, hi = float(np.float32(-30.3 * sy)), float(np.float32(41.7 * sy))      # between codes of the output
    lists = [
        [("clip", lo, hi)],
        [("max", lo), ("clip", -1e6, hi)],
        [("mul", 1.37), ("clip", lo, hi)],
        [("clip", lo, hi), ("mul", 0.5)],
        [("clip", hi, hi)],
        [("clip", 1000 * sy, 2000 * sy)],
        [("clip", -2000 * sy, -1000 * sy)],
        [("add", t) + tq, ("clip", lo, hi)],
        [("mul", 0.7321), ("add", t) + tq, ("mul", 1.25), ("clip", -40 * sy, hi)],
    ]
    xd, wd, bd, td = G.dev(xq), G.dev(wq), G.dev(bq), G.dev(t)
    xp, wp, yp = G.qparams(qp)
    for li, ops in enumerate(lists):
        ref = oracle.qconv2d_chain(xq, qp.x_scale, qp.x_off, wq, qp.w_scale, qp.w_off, bq, ops, qp.y_scale, qp.y_off, (st, st),
                                   (pd,) * 4, g)
        if li == 0:
            assert ref.max() < 127 and ref.min() > -128 and len(np.unique(ref)) > 10, "the bounds do not bind"
        added = any(o[0] == "add" for o in ops)
        for in_place in (False, True) if added else (False,):
            whole, y = G.guarded(yshape, torch.int8)
            if in_place:
                y.copy_(td)
            dev_ops = [("add", y if in_place else td, glowmi.QParam(*tq)) if o[0] == "add" else o for o in ops]
            ws = G.workspace(glowmi.qconv2d_chainv_workspace_bytes(desc, dev_ops))
            glowmi.qconv2d_chainv(xd, xp, wd, wp, bd, y, yp, desc, dev_ops, ws)
            torch.cuda.synchronize()
            variant = glowmi.last_variant()
            what = f"{name} list {li} in place {in_place} [{variant}]"
            assert G.guards_intact(whole, torch.int8), what
            assert variant.endswith("_chainv") and (variant.startswith(kernel) or (added and not adds)), what
            G.assert_equal_i8(y.cpu().numpy(), ref, what)
