"""Python binding of libglowmi.so with the same names as the C ABI (argument marshalling only): the calls that take
tensors go through the native module _native (csrc/python_binding.cpp), which checks the tensors and costs a fraction
of what marshalling them with ctypes does; the structures and the host-side queries are ctypes."""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Tuple

ACT_NONE = 0
ACT_RELU = 1

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libglowmi.so")
_NATIVE_PATH = os.path.join(_HERE, "_native.so")

STATUS_NAMES = {0: "GLOWMI_OK", 1: "GLOWMI_ERR_NULL", 2: "GLOWMI_ERR_SHAPE", 3: "GLOWMI_ERR_UNSUPPORTED",
                4: "GLOWMI_ERR_ALIGN", 5: "GLOWMI_ERR_QUANT", 6: "GLOWMI_ERR_HIP"}


class ConvDesc(ctypes.Structure):
    """glowmi_conv_desc: input n,h,w,c; filter k,r,s; strides; pads (top, left, bottom, right); groups."""
    _fields_ = [(name, ctypes.c_int32) for name in
                ("n", "h", "w", "c", "k", "r", "s", "stride_h", "stride_w",
                 "pad_t", "pad_l", "pad_b", "pad_r", "groups")]


class QParam(ctypes.Structure):
    """glowmi_qparam: value = (q - offset) * scale."""
    _fields_ = [("scale", ctypes.c_float), ("offset", ctypes.c_int32)]


class Chain(ctypes.Structure):
    """glowmi_chain: bias add -> + addend (optional tensor of y's shape) -> act."""
    _fields_ = [("addend", ctypes.c_void_p), ("addend_q", QParam), ("act", ctypes.c_int)]


OP_ADD_TENSOR, OP_MUL_SCALAR, OP_MAX_SCALAR, OP_CLIP = 1, 2, 3, 4
MAX_CHAIN_OPS = 4


class ChainOp(ctypes.Structure):
    """glowmi_chain_op: kind; scalars a, b; tensor operand and (quantized form) its scale/offset."""
    _fields_ = [("kind", ctypes.c_int), ("a", ctypes.c_float), ("b", ctypes.c_float), ("tensor", ctypes.c_void_p),
                ("tensor_q", QParam)]


class SeqLayer(ctypes.Structure):
    """glowmi_seq_layer: one layer of a back-to-back sequence."""
    _fields_ = [("desc", ConvDesc), ("w", ctypes.c_void_p), ("bias", ctypes.c_void_p), ("wq", QParam),
                ("yq", QParam), ("act", ctypes.c_int), ("add_input", ctypes.c_int32)]


class GlowmiError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__(f"{STATUS_NAMES.get(status, status)}: {message}")
        self.status = status


_lib = None
_native = None


def library_path() -> str:
    return _LIB_PATH


def library() -> ctypes.CDLL:
    """Load libglowmi.so and its native binding.  There is no fallback: a missing library is an error."""
    global _lib, _native
    if _lib is not None:
        return _lib
    for path in (_LIB_PATH, _NATIVE_PATH):
        if not os.path.exists(path):
            raise ImportError(f"{path} is missing: build it with `python -m paper_1805_00907_amd.build` "
                              "(glowmi has no CPU or PyTorch fallback)")
    # torch ships its own HIP runtime; import it first so that this library binds to the same
    # runtime instance that owns the device memory and streams handed to it.
    import torch  # noqa: F401
    L = ctypes.CDLL(_LIB_PATH)
    vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
    dp = ctypes.POINTER(ConvDesc)
    L.glowmi_conv_out_shape.argtypes = [dp, ctypes.POINTER(i32), ctypes.POINTER(i32)]
    L.glowmi_conv2d.argtypes = [vp, vp, vp, vp, dp, ctypes.c_int, vp, sz, vp]
    L.glowmi_conv2d_workspace_bytes.argtypes = [dp]
    L.glowmi_conv2d_workspace_bytes.restype = sz
    L.glowmi_fc.argtypes = [vp, vp, vp, vp, i32, i32, i32, ctypes.c_int, vp, sz, vp]
    L.glowmi_fc_workspace_bytes.argtypes = [i32, i32, i32]
    L.glowmi_fc_workspace_bytes.restype = sz
    L.glowmi_fc_noalloc.argtypes = [vp, vp, vp, vp, i32, i32, i32, ctypes.c_int, vp]
    L.glowmi_conv2d_filter_planes_bytes.argtypes = [dp]
    L.glowmi_conv2d_filter_planes_bytes.restype = sz
    L.glowmi_conv2d_pack_filter.argtypes = [vp, dp, vp, sz, vp]
    L.glowmi_conv2d_packed_workspace_bytes.argtypes = [dp]
    L.glowmi_conv2d_packed_workspace_bytes.restype = sz
    L.glowmi_fc_filter_planes_bytes.argtypes = [i32, i32]
    L.glowmi_fc_filter_planes_bytes.restype = sz
    L.glowmi_fc_pack_filter.argtypes = [vp, i32, i32, vp, sz, vp]
    L.glowmi_fc_packed_workspace_bytes.argtypes = [i32, i32, i32]
    L.glowmi_fc_packed_workspace_bytes.restype = sz
    L.glowmi_fc_packed.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, ctypes.c_int, vp, sz, vp]
    L.glowmi_fc_noalloc_max_scratch_bytes.argtypes = []
    L.glowmi_fc_noalloc_max_scratch_bytes.restype = sz
    L.glowmi_tuning_set.argtypes = [ctypes.c_char_p, i32]
    L.glowmi_tuning_reset.argtypes = []
    L.glowmi_tuning_reset.restype = None
    L.glowmi_qconv2d.argtypes = [vp, QParam, vp, QParam, vp, vp, QParam, dp, ctypes.c_int, vp, sz, vp]
    L.glowmi_qconv2d_workspace_bytes.argtypes = [dp]
    L.glowmi_qconv2d_workspace_bytes.restype = sz
    L.glowmi_qfc.argtypes = [vp, QParam, vp, QParam, vp, vp, QParam, i32, i32, i32, ctypes.c_int, vp, sz, vp]
    L.glowmi_qfc_workspace_bytes.argtypes = [i32, i32, i32]
    L.glowmi_qfc_workspace_bytes.restype = sz
    cp = ctypes.POINTER(Chain)
    L.glowmi_conv2d_chain.argtypes = [vp, vp, vp, vp, dp, cp, vp, sz, vp]
    L.glowmi_qconv2d_chain.argtypes = [vp, QParam, vp, QParam, vp, vp, QParam, dp, cp, vp, sz, vp]
    L.glowmi_conv2d_packed.argtypes = [vp, vp, vp, vp, vp, dp, cp, vp, sz, vp]
    op = ctypes.POINTER(ChainOp)
    L.glowmi_conv2d_chainv.argtypes = [vp, vp, vp, vp, dp, op, i32, vp, sz, vp]
    L.glowmi_conv2d_chainv_workspace_bytes.argtypes = [dp, op, i32]
    L.glowmi_conv2d_chainv_workspace_bytes.restype = sz
    L.glowmi_qconv2d_chainv.argtypes = [vp, QParam, vp, QParam, vp, vp, QParam, dp, op, i32, vp, sz, vp]
    L.glowmi_qconv2d_chainv_workspace_bytes.argtypes = [dp, op, i32]
    L.glowmi_qconv2d_chainv_workspace_bytes.restype = sz
    sp = ctypes.POINTER(SeqLayer)
    L.glowmi_seq_arena_bytes.argtypes = [sp, i32, i32]
    L.glowmi_seq_arena_bytes.restype = sz
    L.glowmi_seq_conv2d.argtypes = [vp, sp, i32, vp, vp, sz, vp]
    L.glowmi_seq_qconv2d.argtypes = [vp, QParam, sp, i32, vp, vp, sz, vp]
    L.glowmi_quantize.argtypes = [vp, vp, sz, QParam, vp]
    L.glowmi_dequantize.argtypes = [vp, vp, sz, QParam, vp]
    L.glowmi_rescale.argtypes = [vp, QParam, vp, QParam, sz, vp]
    L.glowmi_fold_batchnorm.argtypes = [vp] * 6 + [ctypes.c_float, i32, ctypes.c_int64, vp, vp]
    L.glowmi_requant_params.argtypes = [ctypes.c_float] * 3 + [ctypes.POINTER(i32)] * 2
    L.glowmi_rescale_params.argtypes = [ctypes.c_float] * 3 + [ctypes.POINTER(i32)] * 2
    L.glowmi_status_string.argtypes = [ctypes.c_int]
    L.glowmi_status_string.restype = ctypes.c_char_p
    L.glowmi_last_error.restype = ctypes.c_char_p
    L.glowmi_last_variant.restype = ctypes.c_char_p
    from . import _native as native      # linked against the library just loaded
    native.structure_types(ConvDesc, QParam, SeqLayer)
    _native = native
    _lib = L
    return L


def _calls():
    """The native entry points (loads the library on first use)."""
    if _native is None:
        library()
    return _native


def _check(status: int) -> None:
    if status != 0:
        raise GlowmiError(status, library().glowmi_last_error().decode())


def last_variant() -> str:
    return library().glowmi_last_variant().decode()


def _conv_counts(desc: ConvDesc) -> Tuple[int, int, int]:
    """(input, filter, output) element counts of a descriptor; zeros when the library will reject it."""
    oh, ow = ctypes.c_int32(0), ctypes.c_int32(0)
    if library().glowmi_conv_out_shape(ctypes.byref(desc), ctypes.byref(oh), ctypes.byref(ow)) != 0:
        return 0, 0, 0
    return (desc.n * desc.h * desc.w * desc.c, desc.k * desc.r * desc.s * (desc.c // desc.groups),
            desc.n * oh.value * ow.value * desc.k)


def conv_out_shape(desc: ConvDesc) -> Tuple[int, int]:
    oh, ow = ctypes.c_int32(0), ctypes.c_int32(0)
    _check(library().glowmi_conv_out_shape(ctypes.byref(desc), ctypes.byref(oh), ctypes.byref(ow)))
    return oh.value, ow.value


def conv2d_workspace_bytes(desc: ConvDesc) -> int:
    return int(library().glowmi_conv2d_workspace_bytes(ctypes.byref(desc)))


def conv2d(x, w, bias, y, desc: ConvDesc, act: int = ACT_NONE, workspace=None, stream=None) -> None:
    _check(_calls().conv2d_packed(x, w, None, bias, y, desc, None, act, workspace, stream))


def fc_workspace_bytes(M: int, K: int, N: int) -> int:
    return int(library().glowmi_fc_workspace_bytes(M, K, N))


def fc(a, w, bias, y, M: int, K: int, N: int, act: int = ACT_NONE, workspace=None, stream=None) -> None:
    _check(_calls().fc_packed(a, w, None, bias, y, M, K, N, act, workspace, stream))


def fc_noalloc(a, w, bias, y, M: int, K: int, N: int, act: int = ACT_NONE, stream=None) -> None:
    """glowmi_fc without a workspace argument and without any allocation (library-owned static scratch)."""
    _check(_calls().fc_noalloc(a, w, bias, y, M, K, N, act, stream))


def fc_noalloc_max_scratch_bytes() -> int:
    return int(library().glowmi_fc_noalloc_max_scratch_bytes())


def tuning_set(name: str, value: int) -> None:
    """Set a tuning knob (experiments and tests), e.g. tuning_set("F32_TILE", 2)."""
    _check(library().glowmi_tuning_set(name.encode(), int(value)))


def tuning_reset() -> None:
    """Every knob back to the planner's own choice."""
    library().glowmi_tuning_reset()


def qconv2d_workspace_bytes(desc: ConvDesc) -> int:
    return int(library().glowmi_qconv2d_workspace_bytes(ctypes.byref(desc)))


def qconv2d(x, xq: QParam, w, wq: QParam, bias, y, yq: QParam, desc: ConvDesc, act: int = ACT_NONE,
            workspace=None, stream=None) -> None:
    _check(_calls().qconv2d_chain(x, xq, w, wq, bias, y, yq, desc, None, None, act, workspace, stream))


def conv2d_chain(x, w, bias, y, desc: ConvDesc, addend=None, act: int = ACT_NONE, workspace=None,
                 stream=None) -> None:
    """y = act(conv + bias + addend); addend is a float tensor of y's shape (may be y) or None."""
    _check(_calls().conv2d_packed(x, w, None, bias, y, desc, addend, act, workspace, stream))


def conv2d_filter_planes_bytes(desc: ConvDesc) -> int:
    return int(library().glowmi_conv2d_filter_planes_bytes(ctypes.byref(desc)))


def conv2d_pack_filter(w, desc: ConvDesc, planes, stream=None) -> None:
    """Writes the fp16 planes of the filter `w` (made once, ahead of the calls that use them) to `planes`."""
    _check(_calls().conv2d_pack_filter(w, desc, planes, stream))


def conv2d_packed_workspace_bytes(desc: ConvDesc) -> int:
    return int(library().glowmi_conv2d_packed_workspace_bytes(ctypes.byref(desc)))


def conv2d_packed(x, w, w_planes, bias, y, desc: ConvDesc, addend=None, act: int = ACT_NONE, workspace=None,
                  stream=None) -> None:
    """conv2d_chain with the filter's planes from conv2d_pack_filter (None: the plain call)."""
    _check(_calls().conv2d_packed(x, w, w_planes, bias, y, desc, addend, act, workspace, stream))


def fc_filter_planes_bytes(K: int, N: int) -> int:
    return int(library().glowmi_fc_filter_planes_bytes(K, N))


def fc_pack_filter(w, K: int, N: int, planes, stream=None) -> None:
    """Writes the fp16 planes of the [K][N] weight `w` (transposed to [N][K]) to `planes`."""
    _check(_calls().fc_pack_filter(w, K, N, planes, stream))


def fc_packed_workspace_bytes(M: int, K: int, N: int) -> int:
    return int(library().glowmi_fc_packed_workspace_bytes(M, K, N))


def fc_packed(a, w, w_planes, bias, y, M: int, K: int, N: int, act: int = ACT_NONE, workspace=None,
              stream=None) -> None:
    """fc with the weight's planes from fc_pack_filter (None: the plain call)."""
    _check(_calls().fc_packed(a, w, w_planes, bias, y, M, K, N, act, workspace, stream))


def qconv2d_chain(x, xq: QParam, w, wq: QParam, bias, y, yq: QParam, desc: ConvDesc, addend=None,
                  addend_q: Optional[QParam] = None, act: int = ACT_NONE, workspace=None, stream=None) -> None:
    """Quantized form: addend is an int8 tensor of y's shape with scale/offset addend_q."""
    _check(_calls().qconv2d_chain(x, xq, w, wq, bias, y, yq, desc, addend, addend_q, act, workspace, stream))


def chain_ops(ops, dtype: str = "float32", count: Optional[int] = None):
    """ctypes array of ChainOp from a list of ("add", tensor[, QParam]) | ("mul", a) | ("max", a) |
    ("clip", a, b).  Tensors are device tensors of the output's element type (or raw addresses)."""
    arr = (ChainOp * max(1, len(ops)))()
    for i, o in enumerate(ops):
        if o[0] == "add":
            q = o[2] if len(o) > 2 else QParam(1.0, 0)
            arr[i] = ChainOp(OP_ADD_TENSOR, 0.0, 0.0, _calls().address(o[1], dtype, count, f"op {i} tensor"), q)
        elif o[0] == "mul":
            arr[i] = ChainOp(OP_MUL_SCALAR, o[1], 0.0, None, QParam(1.0, 0))
        elif o[0] == "max":
            arr[i] = ChainOp(OP_MAX_SCALAR, o[1], 0.0, None, QParam(1.0, 0))
        elif o[0] == "clip":
            arr[i] = ChainOp(OP_CLIP, o[1], o[2], None, QParam(1.0, 0))
        else:
            raise ValueError(f"unknown chain op {o[0]!r}")
    return arr


def conv2d_chainv_workspace_bytes(desc: ConvDesc, ops) -> int:
    arr = chain_ops(ops)
    return int(library().glowmi_conv2d_chainv_workspace_bytes(ctypes.byref(desc), arr, len(ops)))


def conv2d_chainv(x, w, bias, y, desc: ConvDesc, ops, workspace=None, stream=None) -> None:
    """y = ops applied in order to (conv + bias): a general stack of data-parallel operators."""
    _check(_calls().conv2d_chainv(x, w, bias, y, desc, ops, workspace, stream))


def qconv2d_chainv_workspace_bytes(desc: ConvDesc, ops) -> int:
    arr = chain_ops(ops, "int8")
    return int(library().glowmi_qconv2d_chainv_workspace_bytes(ctypes.byref(desc), arr, len(ops)))


def qconv2d_chainv(x, xq: QParam, w, wq: QParam, bias, y, yq: QParam, desc: ConvDesc, ops, workspace=None,
                   stream=None) -> None:
    """Quantized general chain: the ops act on the int32 accumulator, then one requantize."""
    _check(_calls().qconv2d_chainv(x, xq, w, wq, bias, y, yq, desc, ops, workspace, stream))


def qfc_workspace_bytes(M: int, K: int, N: int) -> int:
    return int(library().glowmi_qfc_workspace_bytes(M, K, N))


def qfc(a, aq: QParam, w, wq: QParam, bias, y, yq: QParam, M: int, K: int, N: int, act: int = ACT_NONE,
        workspace=None, stream=None) -> None:
    _check(_calls().qfc(a, aq, w, wq, bias, y, yq, M, K, N, act, workspace, stream))


def requant_params(x_scale: float, w_scale: float, y_scale: float) -> Tuple[int, int]:
    m, s = ctypes.c_int32(0), ctypes.c_int32(0)
    _check(library().glowmi_requant_params(x_scale, w_scale, y_scale, ctypes.byref(m), ctypes.byref(s)))
    return m.value, s.value


def rescale_params(r_scale: float, x_scale: float, w_scale: float) -> Tuple[int, int]:
    m, s = ctypes.c_int32(0), ctypes.c_int32(0)
    _check(library().glowmi_rescale_params(r_scale, x_scale, w_scale, ctypes.byref(m), ctypes.byref(s)))
    return m.value, s.value


def quantize(x, q, qp: QParam, count: Optional[int] = None, stream=None) -> None:
    """float32 device tensor x -> int8 device tensor q with scale/offset qp."""
    _check(_calls().quantize(x, q, qp, count, stream))


def dequantize(q, x, qp: QParam, count: Optional[int] = None, stream=None) -> None:
    _check(_calls().dequantize(q, x, qp, count, stream))


def rescale(q_in, from_q: QParam, q_out, to_q: QParam, count: Optional[int] = None, stream=None) -> None:
    """The same real values on another scale/offset; q_out may be q_in."""
    _check(_calls().rescale(q_in, from_q, q_out, to_q, count, stream))


def fold_batchnorm(w, bias, gamma, beta, mean, var, eps: float):
    """Host arrays (numpy float32): -> (w_folded, bias_folded) with batch normalization merged in."""
    import numpy as np
    w = np.ascontiguousarray(w, dtype=np.float32)
    k = w.shape[0]
    per = w.size // k
    arrs = [None if a is None else np.ascontiguousarray(a, dtype=np.float32) for a in (bias, gamma, beta, mean, var)]
    w_out, b_out = np.empty_like(w), np.empty((k,), dtype=np.float32)
    hp = lambda a: None if a is None else a.ctypes.data
    _check(library().glowmi_fold_batchnorm(hp(w), hp(arrs[0]), hp(arrs[1]), hp(arrs[2]), hp(arrs[3]), hp(arrs[4]),
                                           eps, k, per, hp(w_out), hp(b_out)))
    return w_out, b_out


def seq_layers(layers) -> "ctypes.Array":
    """ctypes array of SeqLayer from (desc, w, bias, act, add_input[, wq, yq]) tuples of device tensors."""
    arr = (SeqLayer * len(layers))()
    for i, l in enumerate(layers):
        desc, w, bias, act, add_input = l[:5]
        quantized = len(l) > 5
        wq, yq = (l[5], l[6]) if quantized else (QParam(1.0, 0), QParam(1.0, 0))
        _, nw, _ = _conv_counts(desc)
        arr[i] = SeqLayer(desc, _calls().address(w, "int8" if quantized else "float32", nw, f"layer {i} w"),
                          _calls().address(bias, "int32" if quantized else "float32", desc.k, f"layer {i} bias"), wq, yq, act,
                          1 if add_input else 0)
    return arr


def seq_arena_bytes(arr, quantized: bool) -> int:
    return int(library().glowmi_seq_arena_bytes(arr, len(arr), 1 if quantized else 0))


def seq_conv2d(x, arr, y, arena, stream=None) -> None:
    _check(_calls().seq_conv2d(x, arr, y, arena, stream))


def seq_qconv2d(x, xq: QParam, arr, y, arena, stream=None) -> None:
    _check(_calls().seq_qconv2d(x, xq, arr, y, arena, stream))
