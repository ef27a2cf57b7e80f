"""Compile libdaspmm.so (HIP kernels + C ABI) for gfx950 and the Python module _native on top of it, in-tree,
with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libdaspmm.so")
SOURCES = ["da_spmm_api.hip", "da_spmm_select.cpp"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-munsafe-fp-atomics",
    # packed fp32 arithmetic stays off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def build_hip(verbose: bool = False) -> str:
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), *FLAGS, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-o", tmp,
           *[os.path.join(CSRC, s) for s in SOURCES]]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    os.replace(tmp, LIB)
    build_native(verbose)
    return LIB


NATIVE = os.path.join(PKG, "_native.so")


def build_native(verbose: bool = False) -> str:
    """The Python module _native (host code only), linked against libdaspmm.so beside it and the
    torch libraries of the running interpreter."""
    import sysconfig

    import torch
    tdir = os.path.dirname(os.path.abspath(torch.__file__))
    tmp = NATIVE + ".tmp%d" % os.getpid()
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc())))
    cmd = [hipcc(), "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
           "-isystem", os.path.join(rocm, "include"), "-DTORCH_EXTENSION_NAME=_native",
           "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"],
           "-isystem", os.path.join(tdir, "include"), "-isystem", os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
           os.path.join(CSRC, "native.cpp"), "-o", tmp,
           "-L" + PKG, "-ldaspmm", "-L" + os.path.join(tdir, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu",
           "-ltorch_hip", "-lc10", "-lc10_hip", "-lamdhip64", "-L" + os.path.join(rocm, "lib"), "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + os.path.join(tdir, "lib")]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout)
    os.replace(tmp, NATIVE)
    return NATIVE


CALIB = os.path.join(PKG, "calib_copy")
CEILINGS = os.path.join(PKG, "ceilings")


def _build_tool(src: str, exe: str, verbose: bool) -> str:
    cmd = [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-munsafe-fp-atomics",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-o", exe, os.path.join(CSRC, src)]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout)
    return exe


def build_calib(verbose: bool = False) -> str:
    """Stand-alone measurement tools: the copy kernel that calibrates rocprofv3's HBM traffic
    counters, and the stream / gather / atomics ceilings of the memory system."""
    _build_tool("calib_copy.hip", CALIB, verbose)
    return _build_tool("ceilings.hip", CEILINGS, verbose)


if __name__ == "__main__":
    print(build_hip(verbose=True))
    print(build_calib(verbose=True))
