"""Builds libooco.so (HIP kernels + C ABI) for gfx950 with hipcc, and the native half of the Python binding, in-tree.

    python -m paper_2511_21862_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libooco.so")
SOURCES = ["ooco_abi.hip", "ooco_kernels.hip", "ooco_model.hip", "ooco_sort.hip"]
HEADERS = [os.path.join(CSRC, "ooco_internal.h"), os.path.join(HERE, "..", "include", "ooco.h"), os.path.join(CSRC, "ooco_arith.h")]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # never let the compiler form packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]

MARSHAL = os.path.join(HERE, "_binding.so")
MARSHAL_SRC = os.path.join(CSRC, "ooco_py.cpp")


def built_for(torch) -> str:
    """What the marshalling module is compiled against, whose objects it reads directly (numpy checks its version by itself)."""
    return f"ooco_binding for torch {torch.__version__}, python {sys.version_info[0]}.{sys.version_info[1]}"


def has_stamp(path: str, stamp: str) -> bool:
    with open(path, "rb") as f:
        return stamp.encode() + b"\0" in f.read()


def build_marshalling(force: bool = True, verbose: bool = False) -> str | None:
    """The binding's native argument marshalling (host code against this Python, numpy and torch); without torch the
    binding is used for host functions only and does without."""
    try:
        import numpy
        import torch
    except ImportError:
        return None
    stamp = built_for(torch)
    if not force and os.path.exists(MARSHAL) and has_stamp(MARSHAL, stamp):
        if os.path.getmtime(MARSHAL) >= max(os.path.getmtime(f) for f in [MARSHAL_SRC, HEADERS[1]]):
            return MARSHAL
    tinc, tlib = (os.path.join(os.path.dirname(torch.__file__), d) for d in ("include", "lib"))
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f'-DOOCO_BUILT_FOR="{stamp}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    for d in (tinc, os.path.join(tinc, "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"], numpy.get_include(),
              "/opt/rocm/include"):
        cmd += ["-isystem", d]
    cmd += ["-I", os.path.join(HERE, "..", "include"), "-Wall", "-o", MARSHAL, MARSHAL_SRC,
            "-L", tlib, "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n{res.stderr}\n{res.stdout}")
    return MARSHAL


def build_library(force: bool = True, verbose: bool = False) -> str:
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    if not force and os.path.exists(LIB):
        newest = max(os.path.getmtime(f) for f in srcs + HEADERS)
        if os.path.getmtime(LIB) >= newest:
            return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + ["-I", os.path.join(HERE, "..", "include"), "-o", LIB] + srcs
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 feature: harmless, filtered
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed:\n{err}\n{res.stdout}")
    if err.strip() and verbose:
        print(err, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build_library(force=True, verbose=True))
    print(build_marshalling(force=True, verbose=True))
