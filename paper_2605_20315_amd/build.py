"""Build libmixquant.so (HIP, gfx950, with hipcc) and the native part of the torch binding (host code, with the C++
compiler) in-tree.  Run as ``python -m paper_2605_20315_amd.build``."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmixquant.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["api.hip", "quantize.hip", "gemm.hip"]
CXX = os.environ.get("CXX", "g++")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",                      # the quantizer's FP32 steps must stay unfused
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def build_library(verbose: bool = False) -> str:
    """Compile every HIP source into one shared library; always recompiles."""
    cmd = [HIPCC] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    noise = "packed-fp32-ops"
    err = "\n".join(l for l in proc.stderr.splitlines() if noise not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    os.replace(LIB + ".tmp", LIB)
    return LIB


def build_binding(verbose: bool = False) -> str:
    """Compile csrc/binding.cpp into the extension module that ops.py calls first; always recompiles."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    includes = [f for d in cpp_extension.include_paths("cuda") + [sysconfig.get_paths()["include"]] for f in ("-isystem", d)]
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", *includes,
           os.path.join(CSRC, "binding.cpp"), "-o", BINDING + ".tmp",
           "-L" + libs, "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("the C++ compiler failed:\n" + proc.stderr)
    if verbose and proc.stderr.strip():
        print(proc.stderr, file=sys.stderr)
    os.replace(BINDING + ".tmp", BINDING)
    return BINDING


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_binding(verbose=True))
