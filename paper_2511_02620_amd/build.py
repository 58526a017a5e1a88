"""Build libdifr.so (HIP kernels + C ABI) for gfx950 with hipcc, and _native.so (the Python side of the C ABI) with the
host compiler, in-tree.

``python -m paper_2511_02620_amd.build`` compiles every source under ``csrc/`` and links
``paper_2511_02620_amd/libdifr.so`` and ``paper_2511_02620_amd/_native.so``.  Nothing is built at import time: tests, the smoke check and
the benchmark load what this step left behind.
"""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdifr.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["api.hip", "gumbel.hip", "ipt.hip", "fused.hip", "split.hip", "likelihood.hip", "ipt_filtered.hip", "nucleus.hip", "lmhead.hip", "reduce.hip"]

# -packed-fp32-ops is switched off: the compiler must not form packed fp32 instructions.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-Wall",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc()] + HIPCC_FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, proc.stdout))
    noise = "'-packed-fp32-ops' is not a recognized feature"
    out = "\n".join(l for l in proc.stdout.splitlines() if noise not in l and l.strip())
    if out:
        sys.stderr.write(out + "\n")
    return obj


def _build_native() -> None:
    import torch

    home = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(hipcc()))
    tmp = NATIVE + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"]
    for d in (os.path.join(home, "include"), os.path.join(home, "include", "torch", "csrc", "api", "include"),
              os.path.join(rocm, "include"), sysconfig.get_paths()["include"]):
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "binding.cpp"), "-o", tmp, "-L" + os.path.join(home, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu",
            "-ltorch_hip", "-ltorch_python"]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode:
        raise RuntimeError("the host compiler failed for binding.cpp:\n%s" % proc.stdout)
    if proc.stdout.strip():
        sys.stderr.write(proc.stdout)
    os.replace(tmp, NATIVE)


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=5) as pool:
        native = pool.submit(_build_native)
        objs = list(pool.map(_compile, SOURCES))
        native.result()
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-o", tmp] + objs
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode:
        raise RuntimeError("link failed:\n%s" % proc.stdout)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
