"""Build libw4a8.so for gfx950 with hipcc (in-tree, no JIT cache).

Every HIP source is compiled with packed-fp32 instruction generation turned
off (the MFMA/int paths never need it and the epilogue's fp32 arithmetic is
kept to plain scalar instructions).
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libw4a8.so")
SOURCES = ["quantize.hip", "pack.hip", "gemm_smallm.hip", "gemm_largem.hip", "gemm_largem_group.hip",
           "attention.hip", "flow.hip", "noalloc.hip", "api.cpp"]
# per-source extra flags: the group-scale GEMM instances use VGPR-form MFMAs
EXTRA_FLAGS = {"gemm_largem_group.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", INCLUDE, "-I", CSRC]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    return obj


# measured HBM-read and INT8-MFMA ceilings for the benchmark (not the layer)
CEILING_SOURCES = ["ceiling.hip"]
CEILING_LIB = os.path.join(PKG, "libw4a8_ceiling.so")


# the binding's native fast path: a CPython extension on torch's C++ API
NATIVE_SOURCE = "binding.cpp"
NATIVE_LIB = os.path.join(PKG, "_native.so")


def _build_native() -> None:
    import sysconfig

    import torch

    tdir = os.path.dirname(torch.__file__)
    inc = [INCLUDE, os.path.join(tdir, "include"), os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"], os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include")]
    tlib = os.path.join(tdir, "lib")
    tmp = NATIVE_LIB + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    for i in inc:
        cmd += ["-isystem", i]
    cmd += [os.path.join(CSRC, NATIVE_SOURCE), "-o", tmp, LIB, "-L", tlib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
            "-Wl,-rpath,$ORIGIN", f"-Wl,-rpath,{tlib}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"building {NATIVE_SOURCE} failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, NATIVE_LIB)


def _link(objs, lib):
    tmp = lib + ".tmp"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", f"-Wl,-soname,{os.path.basename(lib)}", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, lib)


def build() -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = SOURCES + CEILING_SOURCES
    with cf.ThreadPoolExecutor(max_workers=min(len(srcs), os.cpu_count() or 4)) as ex:
        objs = dict(zip(srcs, ex.map(_compile, srcs)))
    _link([objs[s] for s in SOURCES], LIB)
    _link([objs[s] for s in CEILING_SOURCES], CEILING_LIB)
    _build_native()
    return LIB


if __name__ == "__main__":
    print(build())
