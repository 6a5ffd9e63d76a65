"""Compile the HIP library in-tree for gfx950 (hipcc cross-compiles without a GPU), and the binding's native wrappers."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
SOURCES = [os.path.join(_PKG, "csrc", n) for n in ("specsteer.hip", "split.hip")]
INCLUDE = os.path.join(_ROOT, "include")
LIBRARY = os.path.join(_PKG, "libspecsteer.so")
CALLS_SOURCE = os.path.join(_PKG, "csrc", "calls.cpp")
CALLS = os.path.join(_PKG, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950",
    # packed-fp32 instructions are switched off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # The logit loads are 16 bytes wide on vector types that promise only element alignment (rows of an odd
    # vocabulary start anywhere).  This states to the compiler what the code relies on -- wide global loads at
    # any element-aligned address are legal on this target (the hardware's unaligned access mode, which the
    # ROCm kernel driver enables) -- instead of leaving it to the toolchain's default for the target.
    "-Xclang", "-target-feature", "-Xclang", "+unaligned-access-mode",
    "-shared", "-fPIC", "-Wl,-rpath,/opt/rocm/lib",
]


def _run(cmd: list, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n{proc.stdout}\n{proc.stderr}")


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _run([hipcc, *HIPCC_FLAGS, "-I", INCLUDE, "-o", LIBRARY, *SOURCES], verbose)
    build_calls(verbose)
    return LIBRARY


def build_calls(verbose: bool = False) -> str:
    """The binding's native wrappers, host code against torch's headers and libraries."""
    import torch
    from torch.utils import cpp_extension

    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    includes = [x for d in (INCLUDE, *cpp_extension.include_paths(), sysconfig.get_paths()["include"]) for x in ("-I", d)]
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *includes, "-o", CALLS, CALLS_SOURCE,
          "-L", lib, "-lc10", "-ltorch_cpu", "-ltorch_python", f"-Wl,-rpath,{lib}"], verbose)
    return CALLS


if __name__ == "__main__":
    print(build(verbose=True))
