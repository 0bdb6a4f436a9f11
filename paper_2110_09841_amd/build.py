"""Build the HIP library libcvp.so for gfx950 (in-tree).

hipcc compiles the kernels and the C-ABI host code; packed FP32 instructions
are disabled for every device compile.
"""
import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libcvp.so")

# (source, part): the operator kernels are compiled in three parts
SOURCES = [("cvp_kernels.hip", 0), ("cvp_kernels.hip", 1), ("cvp_kernels.hip", 2), ("cvp_siddon.hip", None),
           ("cvp_blas.hip", None), ("cvp_nn.hip", None), ("cvp_synth.hip", None), ("cvp_capi.cpp", None)]
JOBS = 4      # compilations at a time
ARCH = os.environ.get("CVP_OFFLOAD_ARCH", "gfx950")

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          "-I" + INCLUDE, "-I" + CSRC]
DEVICE = ["--offload-arch=" + ARCH, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    objs, cmds = [], []
    for src, part in SOURCES:
        path = os.path.join(CSRC, src)
        obj = os.path.join(BUILD, src + ("" if part is None else ".%d" % part) + ".o")
        lang = ["-x", "hip"] if src.endswith(".hip") else []
        define = [] if part is None else ["-DCVP_PART=%d" % part]
        cmds.append(["hipcc"] + lang + define + ["-c", path, "-o", obj] + COMMON + DEVICE)
        objs.append(obj)
    with concurrent.futures.ThreadPoolExecutor(JOBS) as pool:
        list(pool.map(lambda cmd: _run(cmd, verbose), cmds))
    tmp = LIB + ".tmp%d" % os.getpid()
    _run(["hipcc", "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp] + objs, verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
