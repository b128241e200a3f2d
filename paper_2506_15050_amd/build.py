"""Builds libtppo.so (HIP, gfx950) in-tree with hipcc.

Run as ``python -m paper_2506_15050_amd.build``.  The shared library is placed
next to this file, and beside it the Python side of its calls
(csrc/marshal.cpp); the binding loads both from there.
"""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtppo.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = ["plan.hip", "select.hip", "egae.hip", "losses.hip", "head.hip", "head_bwd.hip", "value_head.hip", "diag.hip",
           "batcher.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]


def build(verbose=False, extra=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the gfx target feature and says so; harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    build_marshal(verbose)
    return LIB


def build_marshal(verbose=False):
    """The binding's native half, against the installed torch's headers (host code only)."""
    import torch
    top = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", os.path.join(ROOT, "include"),
           "-isystem", os.path.join(top, "include"), "-isystem", os.path.join(top, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL,
           "-L", os.path.join(top, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-L", HERE, "-l:libtppo.so",
           "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("the binding's native half failed to build:\n" + res.stdout)
    return MARSHAL


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
