"""Builds librace_attn.so (HIP, gfx950) in-tree with hipcc, and the CPython extension _native.so that marshals its hot
calls.  Each translation unit is compiled to an object file in parallel, then linked."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librace_attn.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["race_api.cpp", "simple_kernels.hip", "generic_kernels.hip", "mfma_kernels.hip", "static_scratch.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
]


def _compile(src: str) -> str:
    obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc"] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                    if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def _compile_native() -> str:
    """The extension's object file (host code only: a plain C++ compiler)."""
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    obj = os.path.join(CSRC, "native_binding.o")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I" + os.path.join(ROOT, "include"), "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
           "-c", os.path.join(CSRC, "native_binding.cpp"), "-o", obj]
    subprocess.run(cmd, check=True)
    return obj


def build(verbose: bool = False) -> str:
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        native = ex.submit(_compile_native)
        objs = list(ex.map(_compile, SOURCES))
        native_obj = native.result()
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    import torch
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.run(["g++", "-shared", "-o", NATIVE, native_obj, "-L" + HERE, "-l:librace_attn.so", "-L" + torch_lib, "-ltorch_python", "-ltorch_cpu", "-lc10",
                    "-lc10_hip", "-Wl,-rpath,$ORIGIN"], check=True)
    if verbose:
        print("built", LIB, NATIVE)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
