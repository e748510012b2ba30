"""Build libbifattn.so for gfx950 in-tree with hipcc, and the Python
binding's native part with the host compiler.

    python -m paper_2403_08845_amd.build

Compiles the HIP kernels and the host-side C ABI into
``paper_2403_08845_amd/libbifattn.so``. Packed fp32 VALU instructions are
disabled for all device code. ``_bifattn_bind.so`` beside it (host code only,
against torch's headers) checks the arguments of the per-step calls; without
a host compiler or those headers it is left out, and Python checks them.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libbifattn.so")
SOURCES = [os.path.join(CSRC, "bifattn_kernels.hip"), os.path.join(CSRC, "bifattn_host.cpp")]
BIND_SRC = os.path.join(CSRC, "bifattn_bind.cpp")
BIND = os.path.join(HERE, "_bifattn_bind.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators in ordinary VGPRs: the online-softmax rescale works on
    # them with VALU ops, which cannot address AGPRs.
    "-mllvm", "-amdgpu-mfma-vgpr-form", "-mllvm", "-disable-promote-alloca-to-lds",
    "-Wall", "-Wno-unused-function", f"-I{INCLUDE}", f"-I{CSRC}",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    return "hipcc"


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in (res.stderr or "").splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({res.returncode}):\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)


def _cxx() -> str:
    return os.environ.get("CXX", "g++")


def bind_obstacle() -> str | None:
    """What keeps the binding's native part from being built here, if anything."""
    if shutil.which(_cxx()) is None:
        return f"no host compiler ({_cxx()})"
    try:
        from torch.utils.cpp_extension import include_paths
    except ImportError as e:
        return f"torch is not importable ({e})"
    headers = {os.path.join("torch", "csrc", "autograd", "python_variable.h"): include_paths(),
               "Python.h": [sysconfig.get_paths()["include"]]}
    for name, dirs in headers.items():
        if not any(os.path.exists(os.path.join(d, name)) for d in dirs):
            return f"{name} not found"
    return None


def build_bind(verbose: bool = False) -> str:
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    tmp = BIND + ".tmp"
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(hipcc()) or hipcc())))
    dirs = [INCLUDE, os.path.join(rocm, "include"), sysconfig.get_paths()["include"], *include_paths()]
    cmd = [_cxx(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[f"-I{d}" for d in dirs], BIND_SRC, "-o", tmp,
           *[f"-L{d}" for d in library_paths()], "-ltorch_python", "-ltorch_cpu", "-lc10"]
    _run(cmd, verbose)
    os.replace(tmp, BIND)
    return BIND


def build(verbose: bool = False) -> str:
    tmp = LIB + ".tmp"
    _run([hipcc(), *HIPCC_FLAGS, *SOURCES, "-o", tmp], verbose)
    os.replace(tmp, LIB)
    why = bind_obstacle()
    if why is None:
        build_bind(verbose)
    else:
        print(f"{os.path.basename(BIND)} not built: {why}", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
