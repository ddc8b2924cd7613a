"""Builds libmsrl.so (HIP, gfx950) next to this file: `python -m paper_2210_00882_amd.build`."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmsrl.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
] + os.environ.get("MSRL_EXTRA_FLAGS", "").split()


# Flags for single translation units (by file-name prefix): the fp32 kernels of 256 units, one wave per SIMD.  Their tile
# loops (96 MFMAs per chunk with the activation work between them) are longer than the compiler's limit for loops it
# unrolls on request; not unrolled, the register arrays they index end up in scratch memory.  MFMA results stay in
# vector registers: the accumulation registers hold the layer-1 outputs, and a result there would be copied over
# before its tanh.
_F32_256 = ["-mllvm", "-pragma-unroll-threshold=200000", "-mllvm", "-amdgpu-mfma-vgpr-form"]
PER_FILE = {"inst_l17_": _F32_256, "inst_family_h256_f32_": _F32_256}


def _compile(src: str) -> str:
    name = os.path.basename(src)
    obj = os.path.join(OBJ, name + ".o")
    extra = [f for prefix, fl in PER_FILE.items() if name.startswith(prefix) for f in fl]
    subprocess.check_call([HIPCC, *FLAGS, *extra, "-c", src, "-o", obj], stderr=subprocess.STDOUT)
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        objs = list(pool.map(_compile, sources))
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build(int(sys.argv[1]) if len(sys.argv) > 1 else 8))
