"""Build libspx.so (HIP, gfx950) in-tree with hipcc."""
import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libspx.so")
SOURCES = ["api.hip", "transport.hip", "table_build.hip", "composition.hip", "inversion.hip", "noalloc.hip"]
ARCH = "gfx950"
# Machine-level loop-invariant code motion keeps the polynomials' constants of the FP64 library functions
# and the segments' constants in vector registers across the transport loops and spills them: the FP64
# ballistic kernel took 256 VGPRs and 346 spills (121 and none without), the FP64 walk 23 spills
# at 168 VGPRs (139 and none), the FP32 walk 47 (14, in its instances 8 to 25).
SOURCE_FLAGS = {"transport.hip": ["-mllvm", "-disable-machine-licm"]}

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17", "-Wall",
    # no packed FP32 instructions: plain VALU FP32 everywhere
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a*b+c fuses only within one source expression, never across statements: every inlined
    # copy of a device function rounds the same way, so a particle's history does not
    # depend on which code path (launch shape, wave state) ran it
    "-ffp-contract=on",
]


def hipcc() -> str:
    h = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(h):
        raise RuntimeError("hipcc not found: the ROCm toolchain is required to build libspx")
    return h


def _compile(src: str, extra) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc()] + FLAGS + SOURCE_FLAGS.get(src, []) + list(extra) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def build(verbose: bool = False, extra=()) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(lambda s: _compile(s, extra), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
