"""Build the HIP library for gfx950 with hipcc (cross-compiles without a GPU), and the native argument marshalling of the
Python binding."""
from __future__ import annotations

import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libquamba_ssd.so")
BIND = os.path.join(PKG, "_bind.so")
SOURCES = ["api.hip", "probe.hip", "conv1d.hip", "decode.hip", "decode_q8.hip", "hadamard.hip", "mamba1.hip", "prefill_generic.hip", "prefill_mfma.hip", "prefill_wide.hip", "offline.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -packed-fp32-ops is switched off: some packed fp32 forms have given wrong results on this hardware.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _compile(src: str, force: bool) -> str:
    path = os.path.join(CSRC, src)
    obj = os.path.join(OBJ, src + ".o")
    deps = [path, os.path.join(CSRC, "quamba_internal.h"), os.path.join(ROOT, "include", "quamba_ssd.h")]
    deps += [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".h", ".hpp", ".cuh"))]
    if force or not os.path.exists(obj) or any(os.path.getmtime(d) > os.path.getmtime(obj) for d in deps):
        cmd = [HIPCC] + FLAGS + (["-x", "hip"] if src.endswith(".hip") else []) + ["-c", path, "-o", obj]
        subprocess.check_call(cmd)
    return obj


def _rocm_include() -> str:
    """The directory of HIP's headers: beside the compiler, wherever PATH or a link finds it."""
    hipcc = os.path.realpath(shutil.which(HIPCC) or HIPCC)
    for root in (os.path.dirname(os.path.dirname(hipcc)), os.environ.get("ROCM_PATH", ""), "/opt/rocm"):
        include = os.path.join(root, "include")
        if root and os.path.exists(os.path.join(include, "hip", "hip_runtime.h")):
            return include
    raise FileNotFoundError(f"no hip/hip_runtime.h beside {hipcc}, under ROCM_PATH or /opt/rocm")


def _build_bind(force: bool) -> str | None:
    """The extension module that binding.py calls (host code against torch's headers; torch's libraries are already
    loaded when it is imported).  Without torch there are no tensors to call it with, and nothing is built."""
    if importlib.util.find_spec("torch") is None:
        print("torch is not installed: building the C library alone")
        return None
    import torch
    src, header = os.path.join(CSRC, "bind.cpp"), os.path.join(ROOT, "include", "quamba_ssd.h")
    # what it was compiled against: other releases of either have other layouts
    built_for, stamp = f"Python {sys.version}, torch {torch.__version__}", os.path.join(OBJ, "bind.txt")
    known = os.path.exists(stamp) and open(stamp).read() == built_for
    if (force or not known or not os.path.exists(BIND) or
            any(os.path.getmtime(d) > os.path.getmtime(BIND) for d in (src, header))):
        base = os.path.dirname(torch.__file__)
        cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
               f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + os.path.join(ROOT, "include"),
               "-isystem", sysconfig.get_paths()["include"]]
        for d in (os.path.join(base, "include"), os.path.join(base, "include", "torch", "csrc", "api", "include"),
                  _rocm_include()):
            cmd += ["-isystem", d]
        cmd += [src, "-o", BIND, "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
        subprocess.check_call(cmd)
        with open(stamp, "w") as f:
            f.write(built_for)
    return BIND


def build_library(force: bool = True, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        bind = ex.submit(_build_bind, force)
        objs = list(ex.map(lambda s: _compile(s, force), SOURCES))
    # the library first: a C program needs no more, also where the extension cannot be built
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    bind.result()
    return LIB


if __name__ == "__main__":
    print(build_library(force="--incremental" not in sys.argv))
