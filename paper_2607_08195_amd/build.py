"""Build libdsmc.so (HIP for gfx950) in-tree with hipcc.

Every translation unit is compiled without floating-point contraction or
fast-math, so each arithmetic operation is a separately rounded IEEE
operation, and with packed-FP32 instructions disabled."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libdsmc.so")
BUILD = os.path.join(HERE, "_build")

SOURCES = ["kernels.hip", "collide.hip", "walls.hip", "dig.hip", "mlp.hip", "api.cpp", "dig_api.cpp", "mlp_api.cpp",
           "mesh.cpp", "mixed.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-ffp-contract=off", "-fno-fast-math",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-result",
         "-I", INCLUDE, "-I", CSRC]
# Loop-invariant constants hoisted out of loops (the coefficients of FP64 sine,
# cosine, logarithm and power) would take all registers of the collide kernel
# and a wave per SIMD of the wall kernel
EXTRA = {f: ["-mllvm", "-disable-machine-licm"] for f in ("collide.hip", "walls.hip")}


def _compile(src, verbose):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", *FLAGS, *EXTRA.get(src, []), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose=False):
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-z,defs", "-o", LIB + ".tmp", *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
