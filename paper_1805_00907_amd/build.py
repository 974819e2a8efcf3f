"""Build libglowmi.so (HIP kernels + C ABI, hipcc for gfx950) and _native.so (its Python binding, host code) in-tree."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libglowmi.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["api.hip", "igemm_f32.hip", "igemm_i8.hip", "igemm_i8_wide.hip", "conv_k3c64_i8.hip", "fc_small_i8.hip", "conv_smallc_f32.hip", "conv_pw_f32.hip", "conv_small_f32.hip", "conv_few_f32.hip", "conv_few_i8.hip", "conv_short_i8.hip", "conv_short_f32.hip", "block_i8.hip", "fc_few_f32.hip", "conv_smallc_i8.hip", "conv_pw_i8.hip", "elementwise.hip", "sequence.hip", "fc_small_f32.hip", "igemm_f32_p3.hip", "conv_k3c64_f32.hip", "conv_k3_f32.hip", "conv_k3v_f32.hip", "conv_dw.hip", "conv_small_i8.hip", "conv_patch_f32.hip", "fc_tiles_f32.hip", "fc_planes_f32.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # packed-fp32 instruction forms are switched off on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _compile(src: str) -> str:
    obj = os.path.join(CSRC, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _native_object() -> str:
    """The Python binding is host code against torch's and Python's headers."""
    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(CSRC, "python_binding.o")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", os.path.join(root, "include"),
           "-isystem", sysconfig.get_paths()["include"], "-isystem", "/opt/rocm/include", "-Wall",
           "-c", os.path.join(CSRC, "python_binding.cpp"), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compiling the Python binding failed:\n{r.stderr}")
    return obj


def _link_native(obj: str) -> None:
    import torch
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [os.environ.get("CXX", "g++"), "-shared", "-o", NATIVE, obj, LIB, f"-L{libs}", "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-lc10_hip", "-Wl,-rpath,$ORIGIN", "-Wl,--no-as-needed"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"linking the Python binding failed:\n{r.stderr}")


def build_library(verbose: bool = True) -> str:
    """Compile every translation unit (in parallel) and link the shared library. Always rebuilds."""
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        native = ex.submit(_native_object)
        objs = list(ex.map(_compile, SOURCES))
        native_obj = native.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-Wl,-soname,libglowmi.so", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    _link_native(native_obj)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build_library()
