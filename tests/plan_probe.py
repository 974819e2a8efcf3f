"""What the planner chooses for a call, on the host: builds plan_probe.cpp against the library and loads it."""
import collections
import ctypes
import os
import subprocess
import tempfile

import paper_1805_00907_amd as glowmi

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.dirname(os.path.abspath(glowmi.__file__))
UNLIMITED = 1 << 36

Plan = collections.namedtuple("Plan", "kernel tile split_k workspace")


class _Raw(ctypes.Structure):
    _fields_ = [("status", ctypes.c_int32), ("kernel", ctypes.c_int32), ("tile", ctypes.c_int32), ("split_k", ctypes.c_int32),
                ("workspace", ctypes.c_uint64)]


class Probe:
    def __init__(self):
        glowmi.library()
        with tempfile.TemporaryDirectory() as tmp:
            so = os.path.join(tmp, "plan_probe.so")
            subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-isystem", "/opt/rocm/include",
                            "-o", so, os.path.join(HERE, "plan_probe.cpp"), os.path.join(PKG, "libglowmi.so"), f"-Wl,-rpath,{PKG}"],
                           check=True, capture_output=True)
            self.lib = ctypes.CDLL(so)
        self.lib.probe_kernel_name.restype = ctypes.c_char_p

    def _plan(self, raw):
        assert raw.status == 0, raw.status
        return Plan(self.lib.probe_kernel_name(raw.kernel).decode(), raw.tile, raw.split_k, raw.workspace)

    def conv(self, desc, quantized=False, addend=False, packed=False, w_offset=0, workspace=UNLIMITED):
        raw = _Raw()
        self.lib.probe_conv(ctypes.byref(desc), int(quantized), int(addend), int(packed), int(w_offset), ctypes.c_uint64(workspace),
                            ctypes.byref(raw))
        return self._plan(raw)

    def conv_versus(self, desc, name, value, packed=False, repeats=400):
        """Median nanoseconds of planning the layer: with that switch, with none."""
        ns = (ctypes.c_int64 * 2)()
        self.lib.probe_conv_versus(ctypes.byref(desc), int(packed), name.encode(), value, repeats, ns)
        return tuple(ns)

    def fc(self, m, k, n):
        raw = _Raw()
        self.lib.probe_fc(m, k, n, ctypes.byref(raw))
        return self._plan(raw)

    def fc_versus(self, m, k, n, name, value, repeats=400):
        ns = (ctypes.c_int64 * 2)()
        self.lib.probe_fc_versus(m, k, n, name.encode(), value, repeats, ns)
        return tuple(ns)

    def qfc(self, m, k, n, w_offset=0):
        raw = _Raw()
        self.lib.probe_qfc(m, k, n, w_offset, ctypes.byref(raw))
        return self._plan(raw)
