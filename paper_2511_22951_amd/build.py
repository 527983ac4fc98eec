"""Build libmd950.so (the HIP kernels and the C ABI of include/md.h) for gfx950.

Each .hip source is compiled separately with hipcc and the objects are linked
into one shared library next to this file.  md_neigh.hip is compiled with
-ffp-contract=off (bit-exact wrap and minimum-image distances).  Packed FP32
instructions are disabled for all device code.
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OUT = os.path.join(HERE, "libmd950.so")
BUILD = os.path.join(HERE, "_build")

SOURCES = ["md_api.hip", "md_neigh.hip", "md_tables.hip", "md_force.hip", "md_verlet.hip",
           "md_adjoint.hip", "md_profile.hip", "md_bpnn.hip"]
# -disable-machine-licm: md_bpnn.hip's loops use more FP64 constants than registers can hold beside
# the accumulators; hoisted out of the loops they spill (98 VGPRs in the symmetry-function kernel of
# the common sets, 32 and more in four others).  Kept in, that kernel spills 4 VGPRs (20 bytes of
# scratch per lane, under its bound of three waves per SIMD) and no other does.  In md_neigh.hip the
# strided list build spills 3 VGPRs without it.
EXTRA = {"md_neigh.hip": ["-ffp-contract=off", "-mllvm", "-disable-machine-licm"],
         "md_bpnn.hip": ["-mllvm", "-disable-machine-licm"]}
ARCH = os.environ.get("MD950_ARCH", "gfx950")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _flags():
    return ["-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH, "-I" + INCLUDE, "-I" + CSRC,
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", "-Wno-unknown-pragmas"]


def _compile(src, verbose):
    obj = os.path.join(BUILD, src.replace(".hip", ".o"))
    cmd = [HIPCC, "-c", "-x", "hip", os.path.join(CSRC, src), "-o", obj] + _flags() + EXTRA.get(src, [])
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", OUT + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    os.replace(OUT + ".tmp", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(OUT)
