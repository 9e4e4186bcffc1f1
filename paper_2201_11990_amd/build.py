"""Compile the gfx950 layer-slice library into paper_2201_11990_amd/libmtnlg.so.

``python -m paper_2201_11990_amd.build`` or :func:`build`.  Each source is compiled
to an object (in parallel), then linked; hipcc cross-compiles without a GPU.
"""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmtnlg.so")
OBJDIR = os.path.join(HERE, "_build")
SOURCES = ("api.cpp", "profile.cpp", "elementwise.hip", "gemm_generic.hip", "gemm_mfma.hip", "gemm_wave.hip", "gemm_parts.hip",
           "attention_f32.hip", "attention_mfma.hip", "attention_fwd16.hip", "attention_bwd.hip", "attention_bwd64.hip", "optimizer.hip", "head.hip", "calibrate.hip")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes"]
# Kernels of four waves may have more than 256 registers, of which the vector unit reads 256.  By default the compiler then puts the results of all matrix
# instructions into the others and copies scores back element by element.
SOURCE_FLAGS = {f: ["-mllvm", "-amdgpu-mfma-vgpr-form=1"] for f in ("attention_mfma.hip", "attention_bwd.hip")}


def _compile(src):
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", *FLAGS, *SOURCE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # expected and harmless: the host pass does not know the packed-fp32 feature; the code generator remarks on M0 in
    # the clobber lists of the LDS-DMA asm statements (csrc/common.h says why it is there)
    quiet = ("packed-fp32-ops", "clobber list contains reserved registers", "Reserved registers on the clobber list")
    err = "\n".join(l for l in res.stderr.splitlines() if not any(q in l for q in quiet))
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        print(err)
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build())
