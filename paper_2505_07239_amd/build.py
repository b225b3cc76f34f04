"""Builds ``libcomet_ring.so`` (hipcc, gfx950 only) and the native part of the binding, ``_host.so`` (g++ against
torch's headers), next to this file."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcomet_ring.so")
HOST = os.path.join(HERE, "_host.so")
# the variants of the matrix-core kernels come first: they take longest to compile
SOURCES = ["ring_gemm_planes_128x64_own.hip", "ring_gemm_group_128x64.hip", "ring_gemm_group_128x64_own.hip",
           "ring_gemm_planes_128x64.hip", "ring_gemm_planes_64x128.hip", "ring_gemm_planes_64x128_listed.hip",
           "ring_gemm_planes_64x64.hip", "ring_gemm_planes_64x64_listed.hip",
           "ring_gemm_planes_32x128.hip", "ring_gemm_planes_32x128_listed.hip",
           "ring_words_64x64.hip", "ring_words_64x64_listed.hip", "ring_tile_32x256.hip", "ring_tile_32x256_listed.hip", "ring_tile_64x64.hip", "ring_tile_64x64_listed.hip",
           "ring_gemm.hip", "wplanes.hip", "ring_skinny.hip", "ring_fewrow.hip", "ctx.hip", "elementwise.hip", "compact.hip",
           "components.hip", "glue.hip", "probe.hip"]
FLAGS = ["-O3", "-std=c++20", "--offload-arch=gfx950", "-fPIC", "-fvisibility=default",
         # the LDS-DMA helper names M0 as clobbered, which clang flags as a reserved register
         "-Wno-inline-asm",
         # packed-FP32 instruction selection is switched off for every device pass
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def rocm() -> str:
    """The ROCm installation whose headers torch's include: ROCM_PATH, or the one that hipcc() belongs to."""
    return os.environ.get("ROCM_PATH") or os.path.dirname(os.path.dirname(hipcc()))


def host_command():
    """The command that builds ``_host.so``: the CPython and torch of the interpreter that runs this."""
    import sysconfig
    import torch
    base = os.path.dirname(torch.__file__)
    include = [os.path.join(base, "include"), os.path.join(base, "include", "torch", "csrc", "api", "include"),
               sysconfig.get_paths()["include"], os.path.join(rocm(), "include"), os.path.join(ROOT, "include")]
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
             "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"] + ["-I" + i for i in include] +
            [os.path.join(CSRC, "host.cpp"), "-o", HOST, "-L" + os.path.join(base, "lib"),
             "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"])


def build(verbose: bool = False, incremental: bool = False) -> str:
    """Compiles every translation unit and links the library.  ``incremental``: skip a unit whose
    object file is newer than its source and every header (development convenience; the default
    compiles everything)."""
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    headers += [os.path.join(ROOT, "include", f) for f in os.listdir(os.path.join(ROOT, "include"))]
    newest_header = max(os.path.getmtime(h) for h in headers)

    def compile_one(src):
        obj = os.path.join(build_dir, src.replace(".hip", ".o"))
        if incremental and os.path.exists(obj) and \
                os.path.getmtime(obj) > max(newest_header, os.path.getmtime(os.path.join(CSRC, src))):
            return obj
        cmd = [hipcc()] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
        if err.strip() and verbose:
            print(err, file=sys.stderr)
        return obj

    def compile_host():
        if incremental and os.path.exists(HOST) and os.path.getmtime(HOST) > max(
                newest_header, os.path.getmtime(os.path.join(CSRC, "host.cpp"))):
            return
        res = subprocess.run(host_command(), capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("g++ failed on host.cpp:\n" + res.stderr)

    # translation units compile side by side (the compilers are subprocesses: threads are enough)
    jobs = max(1, min(len(SOURCES), int(os.environ.get("MAX_JOBS", "0")) or (os.cpu_count() or 1), 8))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        host = pool.submit(compile_host)
        objs = list(pool.map(compile_one, SOURCES))
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    host.result()              # (behind the link: the library works without it)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, incremental="--incremental" in sys.argv))
