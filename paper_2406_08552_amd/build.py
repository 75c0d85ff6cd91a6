"""Builds the C-ABI library ``libdfa.so`` (HIP kernels for gfx950 + host code;
needs hipcc alone) and ``_dfa_binding.so``, the native argument marshalling of
its Python binding (needs g++ and torch's headers).

Both are compiled in-tree; nothing is installed.  Every call of
:func:`build_library` and :func:`build_binding` compiles again, so a changed
source is always picked up.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB_PATH = os.path.join(PKG_DIR, "libdfa.so")
BINDING_PATH = os.path.join(PKG_DIR, "_dfa_binding.so")

SOURCES = ["dfa_kernels.hip", "dfa_short.hip", "dfa_gemm.hip", "dfa_reduce.hip", "dfa_api.cpp", "dfa_search.cpp"]
ARCH = "gfx950"
# Packed fp32 VALU forms are kept out of the device code; the host pass only
# warns that it does not know the feature.
HIPCC_FLAGS = ["-O3", "-std=c++17", "-fPIC", "-shared", f"--offload-arch={ARCH}",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-Wall", "-Wno-unused-function"]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cand = os.path.join(rocm, "bin", "hipcc")
    if os.path.exists(cand):
        return cand
    found = shutil.which("hipcc")
    if not found:
        raise RuntimeError("hipcc not found (set ROCM_PATH)")
    return found


def _compile(cmd: list, path: str, verbose: bool) -> None:
    """Run a compiler command that writes `path` (through a temporary file)."""
    tmp = path + ".tmp"
    cmd = [*cmd, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    log = "\n".join(l for l in (res.stdout + res.stderr).splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed ({res.returncode}):\n{log}")
    if verbose and log.strip():
        print(log, flush=True)
    os.replace(tmp, path)


def build_library(verbose: bool = False) -> str:
    """Compile every source into LIB_PATH and return the path."""
    _compile([hipcc(), *HIPCC_FLAGS, f"-I{INCLUDE}", f"-I{CSRC}", *[os.path.join(CSRC, s) for s in SOURCES]],
             LIB_PATH, verbose)
    return LIB_PATH


def build_binding(verbose: bool = False) -> str:
    """Compile the binding's argument marshalling into BINDING_PATH (host code
    only; its symbols of Python and torch come from the importing process) and
    return the path."""
    import torch
    from torch.utils import cpp_extension
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f"-I{sysconfig.get_paths()['include']}", *[f"-isystem{p}" for p in cpp_extension.include_paths()],
           os.path.join(CSRC, "dfa_binding.cpp"),
           *[f"-L{p}" for p in cpp_extension.library_paths()], "-ltorch_python", "-lc10"]
    _compile(cmd, BINDING_PATH, verbose)
    return BINDING_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_binding(verbose=True))
