"""Build libcompkv.so (HIP for gfx950) in-tree: one hipcc compile per source, then a shared link."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libcompkv.so")
SOURCES = ["api.hip", "stats.hip", "select.hip", "fused.hip", "decode.hip", "step.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    # no packed fp32 instructions anywhere in the library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE,
    "-I", CSRC,
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"hipcc failed: {' '.join(cmd)}")
    return res


HOST_LIB = os.path.join(PKG, "_host.so")


def build_host(verbose: bool = False) -> str:
    """_host.so: the binding's call path in native code (csrc/host.cpp, host code only)."""
    import sysconfig

    from torch.utils import cpp_extension

    tmp = HOST_LIB + f".tmp{os.getpid()}"
    dirs = [d for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"], INCLUDE]]
    libs = cpp_extension.library_paths()
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", *(f"-I{d}" for d in dirs),
          os.path.join(CSRC, "host.cpp"), "-o", tmp, *(f"-L{d}" for d in libs), "-ltorch_python", "-ltorch",
          "-ltorch_cpu", "-lc10"], verbose)
    os.replace(tmp, HOST_LIB)
    return HOST_LIB


TRACE_LIB = os.path.join(PKG, "libcompkv_trace.so")


def build(verbose: bool = False, jobs: int = 4, trace: bool = False) -> str:
    """libcompkv.so, or with trace=True libcompkv_trace.so: the same library with the phase marks of the
    fused step compiled in (-DCOMPKV_PHASE_TRACE; see compkv_phase_trace_set)."""
    out_dir = os.path.join(BUILD, "trace") if trace else BUILD
    lib = TRACE_LIB if trace else LIB
    flags = FLAGS + (["-DCOMPKV_PHASE_TRACE"] if trace else [])
    os.makedirs(out_dir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(out_dir, os.path.splitext(src)[0] + ".o")
        _run([HIPCC, *flags, "-c", os.path.join(CSRC, src), "-o", obj], verbose)
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = lib + f".tmp{os.getpid()}"
    _run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
    os.replace(tmp, lib)
    build_host(verbose)  # (the binding enters either library through it)
    return lib


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv, trace="--trace" in sys.argv))
