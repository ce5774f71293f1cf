"""Builds libhiermoe.so (HIP, gfx950 only) in-tree with hipcc, and _hmcall.so, the binding's native half.  No GPU
is needed to build."""
from __future__ import annotations

import glob
import importlib.util
import os
import shutil
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libhiermoe.so")
PROBE_SRC = os.path.join(PKG, "bench_probe", "stream_probe.hip")   # bench.py's flat-stream reference, not product
PROBE_LIB = os.path.join(PKG, "libhmprobe.so")

CALL_SRC = os.path.join(CSRC, "hm_call.cpp")   # host code against torch's headers
CALL_LIB = os.path.join(PKG, "_hmcall.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fno-gpu-rdc",
    # packed-fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc_path() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: libhiermoe.so cannot be built")


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def call_command(out: str):
    """The compiler call for _hmcall.so; torch is found, not imported."""
    torch_dir = importlib.util.find_spec("torch").submodule_search_locations[0]
    rocm = os.path.dirname(os.path.dirname(hipcc_path()))
    if not os.path.exists(os.path.join(rocm, "include", "hip")):
        rocm = "/opt/rocm"
    include, libs = os.path.join(torch_dir, "include"), os.path.join(torch_dir, "lib")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            "-isystem", include, "-isystem", os.path.join(include, "torch", "csrc", "api", "include"),
            "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
            "-I", os.path.join(ROOT, "include"), "-o", out, CALL_SRC,
            "-L", libs, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def build_library(verbose: bool = False) -> str:
    """Compile every csrc/*.hip into libhiermoe.so, the binding's native half and the benchmark's flat-stream
    probe into libraries of their own; always recompiles."""
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc_path(), *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", tmp, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    tmp = CALL_LIB + ".tmp.%d" % os.getpid()
    cmd = call_command(tmp)
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, CALL_LIB)
    tmp = PROBE_LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc_path(), *HIPCC_FLAGS, "-o", tmp, PROBE_SRC]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, PROBE_LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
