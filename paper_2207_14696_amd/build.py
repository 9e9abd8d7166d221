"""Build the HIP library in-tree for gfx950, and the Python module that calls it per iteration
(``python -m paper_2207_14696_amd.build``)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbifeat.so")
CALLS = os.path.join(HERE, "_calls.so")
OBJDIR = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
    subprocess.check_call([HIPCC, *FLAGS, "-c", src, "-o", obj])
    return obj


def _compile_calls() -> None:
    """csrc/calls.cpp (host code only), against the torch that is installed."""
    import torch
    base = os.path.dirname(torch.__file__)
    tmp = CALLS + f".tmp{os.getpid()}"
    subprocess.check_call([
        os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
        f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DBF_TORCH_VERSION="{torch.__version__}"',
        "-isystem", os.path.join(base, "include"),
        "-isystem", os.path.join(base, "include", "torch", "csrc", "api", "include"),
        "-I", sysconfig.get_path("include"), os.path.join(CSRC, "calls.cpp"), "-o", tmp,
        "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10",
        "-Wl,-rpath," + os.path.join(base, "lib")])
    os.replace(tmp, CALLS)


def build(verbose: bool = False) -> str:
    """Compile every .hip under csrc/, link libbifeat.so, and build _calls.so (always rebuilds)."""
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        calls = ex.submit(_compile_calls)
        objs = list(ex.map(_compile, srcs))
        calls.result()
    tmp = LIB + f".tmp{os.getpid()}"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
