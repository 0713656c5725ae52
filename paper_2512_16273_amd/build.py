"""Builds the C-ABI library `libtslt.so` for gfx950 with hipcc (cross-compiles without a GPU), and, where there are a host
compiler and the headers of torch and Python, `_binding.so`, the fast path of the Python binding."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB_PATH = os.path.join(HERE, "libtslt.so")
BINDING_PATH = os.path.join(HERE, "_binding.so")
BINDING_SOURCE = os.path.join(HERE, "csrc", "binding.cpp")
SOURCES = [os.path.join(HERE, "csrc", "tslt.hip")]
HEADERS = [os.path.join(HERE, "csrc", n) for n in ("common.h", "bins.h", "handover.h", "pow_table.h", "truncate.h", "sample.h", "verify.h", "rowops.h", "rowsample.h", "exp64.h", "tree.h", "wire.h", "stats.h", "calib.h")] + \
          [os.path.join(ROOT, "include", "tslt.h")]


def hipcc_command(out: str = LIB_PATH) -> list:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    return [hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
            # packed-fp32 instructions are kept out of the generated code
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            # loop-invariant code motion after instruction selection: it carries fp64 constants through the tree
            # kernels' loops in vector registers, to the point of spilling (path of 64 trees 44 us with it, 39 without;
            # two trees, every node, 343 and 327)
            "-mllvm", "-disable-machine-licm",
            "-Wall", "-Wno-unused-function",
            "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
            "-o", out] + SOURCES


def built_for() -> str:
    """What `_binding.so` depends on beside its source; the module carries it."""
    import torch
    return f"torch {torch.__version__}, Python {sys.version_info[0]}.{sys.version_info[1]}"


def binding_possible() -> bool:
    import torch
    headers = (os.path.join(os.path.dirname(torch.__file__), "include", "torch", "csrc", "autograd", "python_variable.h"),
               os.path.join(sysconfig.get_paths()["include"], "Python.h"))
    return shutil.which(os.environ.get("CXX", "g++")) is not None and all(os.path.exists(h) for h in headers)


def binding_command(out: str = BINDING_PATH) -> list:
    import torch
    base = os.path.dirname(torch.__file__)
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DTSLT_BUILT_FOR="{built_for()}"',
            "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(base, "include"),
            "-isystem", os.path.join(base, "include", "torch", "csrc", "api", "include"), "-isystem", sysconfig.get_paths()["include"],
            "-o", out, BINDING_SOURCE, "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build_library(verbose: bool = True) -> str:
    commands = [hipcc_command()]
    if binding_possible():
        commands.append(binding_command())
    else:
        print("no host compiler, or no headers of torch or Python: calls go through ctypes", flush=True)
        if os.path.exists(BINDING_PATH):
            os.remove(BINDING_PATH)                    # (of an earlier source, perhaps)
    for cmd in commands:
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    return LIB_PATH


def is_stale() -> bool:
    def older(out, sources):
        return not os.path.exists(out) or any(os.path.exists(s) and os.path.getmtime(s) > os.path.getmtime(out) for s in sources)
    if older(LIB_PATH, SOURCES + HEADERS):
        return True
    if not binding_possible():
        return False
    if older(BINDING_PATH, [BINDING_SOURCE, HEADERS[-1]]):
        return True
    with open(BINDING_PATH, "rb") as f:                # another torch or Python than it was built for
        return built_for().encode() + b"\0" not in f.read()


if __name__ == "__main__":
    build_library()
    print(LIB_PATH)
    sys.exit(0)
