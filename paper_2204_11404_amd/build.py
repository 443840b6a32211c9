"""Build libqecsv.so (HIP for gfx950) in-tree with hipcc."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libqecsv.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # no packed FP32 instructions in any kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]

# object -> (source, macros): the register passes have hundreds of kernel
# instantiations, compiled side by side
PARTS = {"qecsv": ("qecsv.hip", [])}
for _part in range(3):
    for _t in ("float", "double"):
        PARTS["passes_%d_%s" % (_part, _t)] = ("passes.hip", ["-DQEC_PART=%d" % _part, "-DQEC_T=" + _t])


def compile_part(name: str, verbose: bool = False) -> str:
    src, macros = PARTS[name]
    os.makedirs(OBJ, exist_ok=True)
    out = os.path.join(OBJ, name + ".o")
    cmd = [HIPCC, *FLAGS, *macros, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c",
           os.path.join(CSRC, src), "-o", out]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return out


def link(objs, verbose: bool = False) -> str:
    cmd = [HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", *objs, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


def build(verbose: bool = False) -> str:
    workers = max(1, min(len(PARTS), int(os.environ.get("MAX_JOBS") or os.cpu_count() or 1)))
    with ThreadPoolExecutor(workers) as ex:
        objs = list(ex.map(lambda n: compile_part(n, verbose), PARTS))
    return link(objs, verbose)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
