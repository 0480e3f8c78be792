"""Build libmixfp4.so (gfx950) in-tree with hipcc.

Usage: python paper_2605_31035_amd/build.py   (or call build(); importing the
package first would load the library being rebuilt).

Two libraries are built: libmixfp4.so (the C ABI and its kernels) and
_native.so (the binding's native call path, which links it and torch).

Every HIP source is compiled for gfx950 only, with fp contraction off (the
quantizer relies on exact IEEE operations in the order written) and packed
fp32 instructions disabled.  The shared library lands next to this file so
that it travels with the source tree.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmixfp4.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["api.cpp", "quantize.hip", "quantize2d.hip", "dequantize.hip", "gemm.hip",
           "gemm_f16.hip", "gemm_direct.hip", "gemm_route.cpp", "decode_operand.hip",
           "quantize_variant.hip"]

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.path.join(ROCM, "bin", "hipcc")
ARCH = "gfx950"

COMMON = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"),
]


def _run(cmd):
    p = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature; that warning is expected
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in p.stderr.splitlines() if noise not in l)
    if p.returncode != 0:
        raise RuntimeError(f"command failed ({p.returncode}): {' '.join(cmd)}\n{err}")
    return err


def _build_native(obj: str) -> None:
    """Compile csrc/binding.cpp against torch (host code only)."""
    import sysconfig

    import torch
    tdir = os.path.dirname(torch.__file__)
    inc = [os.path.join(tdir, "include"), os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"], os.path.join(ROCM, "include"),
           os.path.join(ROOT, "include")]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
          *[f"-isystem{d}" for d in inc], "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj])


def build(verbose: bool = False) -> str:
    """Compile every source and link libmixfp4.so; return its path."""
    if not os.path.exists(HIPCC):
        raise RuntimeError(f"hipcc not found at {HIPCC}")
    os.makedirs(BUILD, exist_ok=True)
    objs = []

    def compile_one(src):
        obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
        lang = ["-x", "hip"] if src.endswith(".hip") else []
        err = _run([HIPCC, *COMMON, *lang, "-c", os.path.join(CSRC, src), "-o", obj])
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    native_obj = os.path.join(BUILD, "binding.o")
    with ThreadPoolExecutor(len(SOURCES) + 1) as ex:
        native = ex.submit(_build_native, native_obj)
        objs = list(ex.map(compile_one, SOURCES))
        native.result()
    tmp = LIB + ".tmp"
    _run([HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp, *objs,
          f"-Wl,-rpath,{os.path.join(ROCM, 'lib')}"])
    shutil.move(tmp, LIB)
    import torch
    tlib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = NATIVE + ".tmp"
    _run(["g++", "-shared", "-fPIC", "-o", tmp, native_obj, f"-L{HERE}", "-l:libmixfp4.so",
          f"-L{tlib}", "-ltorch_python",
          "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN", f"-Wl,-rpath,{tlib}"])
    shutil.move(tmp, NATIVE)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
