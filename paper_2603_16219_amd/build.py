"""Compile the HIP library in-tree for gfx950 (hipcc cross-compiles without a GPU), and the binding's native wrappers."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sysconfig

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
SOURCES = [os.path.join(_PKG, "csrc", n) for n in ("specsteer.hip", "split.hip")]
INCLUDE = os.path.join(_ROOT, "include")
LIBRARY = os.path.join(_PKG, "libspecsteer.so")
CALLS_SOURCES = [os.path.join(_PKG, "csrc", "calls.cpp"), os.path.join(_PKG, "csrc", "unbound.h"), os.path.join(INCLUDE, "specsteer.h")]

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
    build_library(verbose)
    build_calls(verbose)
    return LIBRARY


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _run([hipcc, *HIPCC_FLAGS, "-I", INCLUDE, "-o", LIBRARY, *SOURCES], verbose)
    return LIBRARY


def calls_path() -> str:
    """Where the native wrappers for this torch and these sources lie: what they are compiled against is in the name, so that one
    built for another torch, whose tensors may be laid out differently, or from other sources is never loaded."""
    import torch

    h = hashlib.sha256(repr((torch.__version__, torch.version.git_version, torch._C._GLIBCXX_USE_CXX11_ABI)).encode())
    for path in CALLS_SOURCES:
        with open(path, "rb") as f:
            h.update(f.read())
    return os.path.join(_PKG, f"_calls-{h.hexdigest()[:16]}{sysconfig.get_config_var('EXT_SUFFIX')}")


def build_calls(verbose: bool = False) -> str:
    """The binding's native wrappers, host code against torch's headers and libraries.  Renamed into place, so that processes that
    build at the same time never load half a file."""
    import torch
    from torch.utils import cpp_extension

    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    includes = [x for d in (INCLUDE, *cpp_extension.include_paths(), sysconfig.get_paths()["include"]) for x in ("-I", d)]
    path = calls_path()
    part = f"{path}.{os.getpid()}"
    try:
        _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden",
              f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *includes, "-o", part, CALLS_SOURCES[0],
              "-L", lib, "-lc10", "-ltorch_cpu", "-ltorch_python", f"-Wl,-rpath,{lib}"], verbose)
        os.replace(part, path)
    finally:
        if os.path.exists(part):
            os.remove(part)
    return path


if __name__ == "__main__":
    print(build(verbose=True))
