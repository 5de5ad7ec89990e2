"""Build libzq.so with hipcc for gfx950 (cross-compiles without a GPU) and _zq_host.so, the binding's native calls, with g++
against the installed torch where that is possible; both in-tree."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libzq.so")
HOST = os.path.join(HERE, "_zq_host.so")

SOURCES = [
    "zq_api.hip",
    "zq_quant_kernels.hip",
    "zq_gemm_dispatch.hip",
    "zq_gemm_direct.hip",
    "zq_gemm_vector.hip",
    "zq_gemm_skinny.hip",
    "zq_gemm_tile.hip",
    "zq_probe.hip",
]

# Packed FP32 instructions are kept off.  The first 14 dwords of a kernel's arguments come in scalar registers that
# the launch fills, instead of through a load from memory that the first address waits for; the GeMM kernels therefore
# list what their first loads need first, as plain values (a struct ends the preloaded run).  Microseconds per launch
# in a replayed graph, weights from memory, without / with: 2048x2048 at 1 token 3.70 / 3.49, 2048x8192 at 27 tokens
# 8.45 / 7.91, 6400x1600 at 5 5.00 / 4.71; blocks of width 1600 to 2048 at 1 to 27 tokens 8 % faster.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=14"]


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _compile(src):
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    extra = os.environ.get("ZQ_EXTRA_HIPCC_FLAGS", "").split()
    cmd = [_hipcc()] + FLAGS + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    return obj


def _build_host():
    import sysconfig

    import torch
    at = torch.__path__[0]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(), "-I" + sysconfig.get_paths()["include"]]
    for inc in (os.path.join(at, "include"), os.path.join(at, "include", "torch", "csrc", "api", "include"),
                os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")):
        cmd += ["-isystem", inc]
    cmd += [os.path.join(CSRC, "zq_host.cpp"), "-o", HOST, "-L" + os.path.join(at, "lib"),
            "-lc10", "-lc10_hip", "-ltorch", "-ltorch_cpu", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("the native binding failed to build:\n%s\n%s" % (r.stdout, r.stderr))


def _try_host():
    """Builds _zq_host.so if g++, Python's headers and a ROCm torch are there.  Without it the binding goes through ctypes, so what
    is missing is said and does not end the build; an old one does not stay."""
    try:
        _build_host()
    except (RuntimeError, ImportError, OSError, AttributeError) as e:
        if os.path.exists(HOST):
            os.remove(HOST)
        print("_zq_host.so is not built, calls will go through ctypes: %s" % e, file=sys.stderr)
        return False
    return True


def build(verbose=False, jobs=6):
    """Compile every source and link libzq.so, and _zq_host.so where it can be; always rebuilds."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        host = ex.submit(_try_host)
        objs = list(ex.map(_compile, SOURCES))
        host.result()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
