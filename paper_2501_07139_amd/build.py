"""Build libfq.so (HIP kernels + C-ABI) for gfx950 and the extension module of the binding, in-tree.

    python paper_2501_07139_amd/build.py
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libfq.so")
BIND = os.path.join(PKG, "_bind" + sysconfig.get_config_var("EXT_SUFFIX"))

SOURCES = ["fq_host.cpp", "fq_api.hip", "fq_gemv.hip", "fq_decode.hip", "fq_skinny.hip", "fq_gemm.hip", "fq_dense.hip", "fq_attn.hip", "fq_rowops.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # leading scalar arguments are preloaded into registers, so a kernel's first loads need no round trip to the argument buffer
    # (older firmware runs the compiler's fallback that loads them)
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *FLAGS, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = ("is not a recognized feature for this target", "argument unused during compilation")
    err = "\n".join(l for l in res.stderr.splitlines() if not any(n in l for n in noise))
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_bind() -> str:
    """The extension module that takes Python calls to libfq's entry points; it loads with torch, whose libraries it names.
    Returns what went wrong: the package works without it, so a host without g++ or torch's headers still builds."""
    if os.path.exists(BIND):
        os.remove(BIND)  # never one that belongs to an older source
    try:
        import torch
    except ImportError as e:
        return str(e)
    root = os.path.dirname(torch.__file__)
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               sysconfig.get_paths()["include"], "/opt/rocm/include", os.path.join(ROOT, "include")]
    cmd = ["g++", "-O2", "-fPIC", "-shared", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DFQ_TORCH_VERSION="{torch.__version__}"', *(f"-I{d}" for d in include),
           os.path.join(CSRC, "fq_bind.cpp"), "-o", BIND, "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu",
           "-lc10", "-lc10_hip"]
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
    except OSError as e:
        return str(e)
    return "" if res.returncode == 0 else "g++ failed on fq_bind.cpp:\n" + res.stderr


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        bind = ex.submit(_build_bind)
        objs = list(ex.map(_compile, SOURCES))
        if bind.result():
            print("the extension module of the binding is not built: " + bind.result(), file=sys.stderr)
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
