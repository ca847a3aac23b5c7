"""Build libsolfp4.so (the C-ABI library) in-tree for gfx950 with hipcc, and
_host.so (the Python binding's native calls, host code linked against it).

    python -m paper_2604_06916_amd.build
"""
from __future__ import annotations

import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libsolfp4.so")
HOST_LIB = os.path.join(PKG, "_host.so")
SOURCES = ["api.hip", "quantize.hip", "gemm.hip", "gemm_small.hip", "gemm_wavek.hip", "mx_quantize.hip",
           "mx_gemm.hip"]
HEADERS = ["device_common.h", "kernels.h", "nvfp4_gemm_common.h"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # one fixed FP32 operation order: no mul+add contraction anywhere (the
    # GEMM epilogue's fma is written explicitly)
    "-ffp-contract=off",
    # export only the C-ABI (marked SOLFP4_API in solfp4.h)
    "-fvisibility=hidden",
    # no packed-FP32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return obj


def _compile_host() -> str:
    """The binding's host code: no device code, so the host compiler."""
    torch_dir = importlib.util.find_spec("torch").submodule_search_locations[0]
    obj = os.path.join(OBJ, "host_binding.o")
    inc = os.path.join(torch_dir, "include")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-I", os.path.join(ROOT, "include"),
           "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-I", sysconfig.get_paths()["include"], "-c", os.path.join(CSRC, "host_binding.cpp"), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on host_binding.cpp:\n{r.stderr}")
    return obj


def _link_host(obj: str) -> None:
    torch_lib = os.path.join(importlib.util.find_spec("torch").submodule_search_locations[0], "lib")
    tmp = HOST_LIB + ".tmp"
    cmd = ["g++", "-shared", obj, "-o", tmp, "-L", PKG, "-l:libsolfp4.so", "-Wl,-rpath,$ORIGIN",
           "-L", torch_lib, "-lc10", "-ltorch_cpu", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, HOST_LIB)


def build(verbose: bool = True) -> str:
    """Compile every source and link libsolfp4.so and _host.so; always rebuilds."""
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        raise RuntimeError("hipcc not found")
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        host = ex.submit(_compile_host)
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    _link_host(host.result())
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
