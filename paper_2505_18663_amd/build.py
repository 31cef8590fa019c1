"""Build libdvdq.so (hipcc, gfx950 only) and the binding's native part in-tree, next to this file."""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdvdq.so")

SOURCES = ["api.hip", "rotate_quant.hip", "w4ax_gemm.hip", "w4a4_fp6_gemm.hip", "w4ax_gemm_wide.hip", "w4ax_gemm_small.hip", "gbs.hip", "bgr.hip", "bench_kernels.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # keep the compiler from forming packed fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep atomics as written: the wave-aggregating rewrite waits for the reply right behind the
    # atomic (vmcnt 0), which would stall the GEMM's load pipeline at every tile draw
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
]


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{res.stdout}\n{res.stderr}")
    return obj


def _build_marshal() -> None:
    """csrc/marshal.cpp: host code only, against the headers and libraries of the Python and torch that will load it (the binding
    does without where they, or a host compiler, are not installed)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    from . import _MARSHAL_PATH
    cxx = os.environ.get("CXX", "g++")
    headers = [os.path.join(sysconfig.get_path("include"), "Python.h"),
               *(os.path.join(cpp_extension.include_paths()[0], "torch", "csrc", h) for h in ("Exceptions.h", "autograd/python_variable.h"))]
    if shutil.which(cxx) is None or not all(map(os.path.exists, headers)):
        print(f"no {cxx} or no headers of this Python and torch: {os.path.basename(_MARSHAL_PATH)} not built, calls go through ctypes")
        return
    tmp = _MARSHAL_PATH + f".tmp{os.getpid()}"
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-cast-function-type",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + sysconfig.get_path("include"),
           *("-isystem" + d for d in cpp_extension.include_paths()), os.path.join(CSRC, "marshal.cpp"), "-o", tmp,
           "-L" + torch_lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed for marshal.cpp:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, _MARSHAL_PATH)


def build_library(verbose: bool = False) -> str:
    """Compile every source and link the shared libraries.  Always rebuilds."""
    os.makedirs(OBJ, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(4, len(SOURCES))) as ex:
        marshal = ex.submit(_build_marshal)
        objs = list(ex.map(_compile, SOURCES))
        marshal.result()
    tmp = LIB + f".tmp{os.getpid()}"
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True)
    sys.exit(0)
