"""Build the gfx950 HIP library (libmdgpu.so) in-tree with hipcc.

All HIP code is compiled for gfx950 only, with packed-FP32 instruction
selection switched off (-target-feature -packed-fp32-ops), and with matrix
products accumulating in vector registers (-amdgpu-mfma-vgpr-form: results in
accumulation registers cost a move each before the vector ALU can read them).
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmdgpu.so")
SOURCES = ["md_kernels.hip", "md_surrogate.hip", "md_api.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-munsafe-fp-atomics", "-mllvm", "-amdgpu-mfma-vgpr-form", "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
         "-Wno-unknown-pragmas"]


def build(verbose=False, extra=()):
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC] + FLAGS + list(extra) + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
