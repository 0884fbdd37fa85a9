"""Builds liblrboost.so (hand-written HIP kernels for gfx950 + the C ABI) with hipcc, and the binding's native marshalling, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblrboost.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
OBJ_DIR = os.path.join(HERE, "_build")
SOURCES = ["api.hip", "gemm_bf16.hip", "gemm_ring32.hip", "gemm_ring64.hip", "gemm_ring64x128.hip", "gemm_ring128.hip", "gemm_joint.hip", "gemm_rows16.hip",
           "gemm_f32.hip", "stream_kernels.hip", "attention.hip", "probe.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def _run(what: str, cmd: list) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{r.stdout}\n{r.stderr}")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
    _run(f"hipcc on {src}", ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj])
    return obj


def _compile_marshal() -> tuple:
    """Host code only: g++ against torch's headers.  Returns the object and the options that link it."""
    import torch
    from torch.utils import cpp_extension

    obj = os.path.join(OBJ_DIR, "marshal.o")
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    dirs = [os.path.join(ROOT, "include"), *cpp_extension.include_paths(), os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]
    _run("g++ on marshal.cpp", ["g++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1",
                                f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *("-I" + d for d in dirs), "-c",
                                os.path.join(CSRC, "marshal.cpp"), "-o", obj])
    return obj, ["-L" + HERE, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN", "-L" + libs, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def build_library(verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, os.cpu_count() or 4)) as ex:
        marshal = ex.submit(_compile_marshal)
        objs = list(ex.map(_compile, SOURCES))
    _run("link", ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    obj, options = marshal.result()      # (the library is there whether or not this compiled)
    _run("link of the marshalling", ["g++", "-shared", "-fPIC", "-o", MARSHAL, obj, *options])
    if verbose:
        print(f"built {LIB}", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build_library()
