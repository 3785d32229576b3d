"""Builds libgear.so, the gfx950 experience-replay library, and _binding.so, the
Python entry of its per-step calls, in-tree.

Usage: python -m paper_2310_05205_amd.build
"""
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libgear.so")
BINDING = os.path.join(PKG, "_binding.so")
SOURCES = ["table.hip", "alloc.hip", "select.hip", "topk.hip", "shard.hip", "collect.hip", "update.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wno-unused-function",
    # Keep the compiler from forming packed fp32 instructions.
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _run(cmd, what, verbose):
    r = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass warns about the device-only target feature; drop that noise.
    msgs = [l for l in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in l]
    if r.returncode != 0:
        raise RuntimeError("building %s failed:\n" % what + "\n".join(msgs))
    if verbose and msgs:
        print("\n".join(msgs), file=sys.stderr)


def build_library(verbose=False):
    """Compile every HIP source into libgear.so (always recompiles)."""
    hipcc = os.environ.get("HIPCC", "hipcc")
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc] + HIPCC_FLAGS + ["-I" + INCLUDE, "-I" + CSRC, "-o", tmp]
    cmd += [os.path.join(CSRC, s) for s in SOURCES]
    _run(cmd, "libgear.so", verbose)
    os.replace(tmp, LIB)
    return LIB


def build_binding(verbose=False):
    """Compile the Python entry of the per-step calls (host code only)."""
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    tmp = BINDING + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I" + INCLUDE, "-I" + sysconfig.get_paths()["include"]]
    cmd += ["-isystem" + p for p in include_paths()]
    cmd += [os.path.join(CSRC, "binding.cpp"), "-o", tmp]
    for p in library_paths():
        cmd += ["-L" + p, "-Wl,-rpath," + p]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10"]
    _run(cmd, "_binding.so", verbose)
    os.replace(tmp, BINDING)
    return BINDING


def build(verbose=False):
    """Compile the library and its Python entry; returns the library's path."""
    build_binding(verbose)
    return build_library(verbose)


if __name__ == "__main__":
    print(build(verbose=True))
