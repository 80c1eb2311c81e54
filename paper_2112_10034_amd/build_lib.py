"""Builds libcox.so (HIP, gfx950) in-tree with hipcc, and _coxbind.so (the
binding's native fast path, host C++ against torch's headers) with g++.

Device code is compiled without floating-point contraction (every binary32
add, multiply and FMA is the one the schedule names), without packed-FP32
instructions, and with denormals preserved.
"""
import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libcox.so")
BIND = os.path.join(HERE, "_coxbind.so")
BUILD = os.path.join(HERE, "_build")

SOURCES = ["capi.hip", "reduce.hip", "scan.hip", "sort.hip", "tile.hip", "stream.hip", "segmented.hip", "dynamic.hip", "grid.hip", "image.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-I", INCLUDE,
]


def _compile(src, verbose):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature; that warning is harmless
    msgs = [ln for ln in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in ln]
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n" + "\n".join(msgs))
    if verbose and msgs:
        print("\n".join(msgs), flush=True)
    return obj


def _compile_bind(verbose):
    import torch

    root = os.path.dirname(torch.__file__)
    inc = os.path.join(root, "include")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "bind.cpp"), "-o", BIND + ".tmp",
           "-L", os.path.join(root, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on bind.cpp:\n" + r.stdout + r.stderr)
    if verbose and r.stderr:
        print(r.stderr, flush=True)
    os.replace(BIND + ".tmp", BIND)


def build(verbose=False, jobs=None):
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(len(SOURCES) + 1, os.cpu_count() or 1, 8)
    with cf.ThreadPoolExecutor(jobs) as ex:
        bind = ex.submit(_compile_bind, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
        try:
            bind.result()
        except Exception as e:  # calls work without it, see cox.py; a stale one must not stay
            if os.path.exists(BIND):
                os.remove(BIND)
            warnings.warn(f"_coxbind.so was not built: {e}")
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB + ".tmp", *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
