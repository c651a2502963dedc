"""Build libfdtd.so (HIP kernels for gfx950 + C++ host runtime) in-tree.

    python -m paper_0802_3775_amd.build [-v]

Every source is compiled with hipcc for gfx950 with floating-point contraction
off (the kernels place their fused multiply-adds explicitly) and without
packed-FP32 instructions.
"""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libfdtd.so")
# (source, extra flags): the step kernels are one file compiled for each tile width
SOURCES = [("step.hip", ["-DFD_STEP_TX=16"]), ("step.hip", ["-DFD_STEP_TX=32"]), ("step.hip", ["-DFD_STEP_TX=64"]),
           ("kernels.hip", []), ("api.cpp", []), ("geometry.cpp", [])]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = ["-O3", "-fPIC", "-std=c++17", "-ffp-contract=off", "-Wall",
          "-I", os.path.join(ROOT, "include"), "-I", CSRC]
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
HOST = ["-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include"]


def build(verbose: bool = False) -> str:
    with tempfile.TemporaryDirectory(prefix="fdtd_build_") as tmp:
        def compile_one(at):
            src, flags = SOURCES[at]
            obj = os.path.join(tmp, "%d_%s.o" % (at, src))
            cmd = [HIPCC] + COMMON + (DEVICE if src.endswith(".hip") else HOST) + flags + \
                  ["-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        with ThreadPoolExecutor(4) as pool:
            objs = list(pool.map(compile_one, range(len(SOURCES))))
        cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB + ".tmp"] + objs
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
