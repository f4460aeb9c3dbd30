"""Build the gfx950 shared library ``libmxfp4_hip.so`` in-tree with hipcc, and the extension module ``_host.so`` of
the binding.

Run ``python -m paper_2503_13565_amd.build``.  hipcc cross-compiles without a GPU.  Object
files go to ``paper_2503_13565_amd/_build/`` (not committed); both land next to this
file so that they travel with the source tree.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmxfp4_hip.so")
HOST = os.path.join(HERE, "_host.so")
SOURCES = ["api.hip", "cast.hip", "gemv.hip", "gemv_reg.hip", "gemv_short.hip", "chain.hip", "mfma.hip", "mfma_tile.hip", "bf16.hip", "e4m3.hip", "e2m3.hip", "mxfmt.hip", "gemm_t.hip", "gemv_tile.hip", "gemm_wide.hip", "gemm_wide_fmt.hip", "gemm_wide_bf16.hip"]
# packed FP32 instructions are disabled on purpose: see the build notes of this project
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# per file: the leading scalar kernel arguments arrive in scalar registers when a wave starts (a cast of 735 x 640 2.79 -> 2.52 us,
# 4008 x 4096 8.2 -> 8.0, 10422 x 7936 36.0 -> 35.9)
PRELOAD = ["-mllvm", "-amdgpu-kernarg-preload-count=16"]
EXTRA = {"gemv_reg.hip": PRELOAD, "gemv_short.hip": PRELOAD, "gemv_tile.hip": PRELOAD, "chain.hip": PRELOAD, "mfma_tile.hip": PRELOAD, "gemv.hip": PRELOAD, "e4m3.hip": PRELOAD, "e2m3.hip": PRELOAD, "mxfmt.hip": PRELOAD, "cast.hip": PRELOAD, "bf16.hip": PRELOAD, "gemm_wide.hip": PRELOAD, "gemm_wide_fmt.hip": PRELOAD, "gemm_wide_bf16.hip": PRELOAD}


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(src: str, verbose: bool, defines=()) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *FLAGS, *EXTRA.get(src, []), *defines, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in proc.stderr.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
    if err.strip() and verbose:
        print(err, file=sys.stderr)
    return obj


def _compile_host(verbose: bool) -> str:
    """The extension module behind the binding: host code against torch's headers."""
    obj, at = os.path.join(BUILD, "host.o"), os.path.join(os.path.dirname(torch.__file__), "include")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DMXFP4_TORCH_VERSION="%s"' % torch.__version__,
           "-isystem", at, "-isystem",
           os.path.join(at, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include", "-isystem",
           sysconfig.get_paths()["include"], "-c", os.path.join(CSRC, "host.cpp"), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("g++ failed on host.cpp:\n%s" % proc.stderr)
    return obj


def _link_host(obj: str, verbose: bool) -> None:
    """Linked against the library beside it, which the binding has loaded by then."""
    tmp, at = HOST + ".tmp.%d" % os.getpid(), os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-shared", "-o", tmp, obj, "-L" + HERE, "-l:" + os.path.basename(LIB), "-L" + at, "-ltorch_python",
           "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, HOST)


def build(verbose: bool = True, jobs: int = 8, knobs: bool = False) -> str:
    """knobs: a measurement build in which the launch-shape switches (environment variables) exist;
    the library as shipped is built without them."""
    os.makedirs(BUILD, exist_ok=True)
    defines = ("-DMXFP4_MEASUREMENT_KNOBS",) if knobs else ()
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        host = ex.submit(_compile_host, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose, defines), SOURCES))
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    _link_host(host.result(), verbose)
    return LIB


if __name__ == "__main__":
    print(build(knobs="--knobs" in sys.argv[1:]))
