"""Builds libsparq.so (HIP, gfx950) in-tree with hipcc, and the native part of the Python binding with g++."""
from __future__ import annotations

import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsparq.so")
PROBE_SRC = os.path.join(CSRC, "probe", "sparq_probe.hip")
PROBE_LIB = os.path.join(HERE, "libsparq_probe.so")   # machine-ceiling micro-benchmarks (include/sparq_probe.h)
NATIVE_SRC = os.path.join(CSRC, "binding", "sparq_native.cpp")
NATIVE_LIB = os.path.join(HERE, "_sparq_native.so")   # argument marshalling of the hot entry points (binding.py)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # keep the compiler from forming packed-fp32 instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
FLAGS += os.environ.get("SPARQ_HIPCC_FLAGS", "").split()


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def build_native() -> str:
    """The binding's extension module: host code against torch's headers, no HIP code in it."""
    import torch
    T = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(HIPCC)))
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", os.path.join(T, "include"),
           "-isystem", os.path.join(T, "include", "torch", "csrc", "api", "include"), "-isystem", os.path.join(rocm, "include"),
           "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"], NATIVE_SRC, "-o", NATIVE_LIB,
           "-L" + os.path.join(T, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on {NATIVE_SRC}:\n{r.stdout}\n{r.stderr}")
    return NATIVE_LIB


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every .hip under csrc/ and link libsparq.so, libsparq_probe.so and _sparq_native.so. Always recompiles."""
    objs = []

    def compile_one(src):
        obj = src[:-4] + ".o"
        cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
        if verbose and r.stderr.strip():
            print(r.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        native = ex.submit(build_native)
        objs = list(ex.map(compile_one, sources()))
        native.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    r = subprocess.run([HIPCC, *FLAGS, "-shared", PROBE_SRC, "-o", PROBE_LIB], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {PROBE_SRC}:\n{r.stdout}\n{r.stderr}")
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
