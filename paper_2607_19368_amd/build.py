"""Build libslh.so (the HIP kernels and the C ABI) for gfx950 with hipcc.

    python -m paper_2607_19368_amd.build        # or paper_2607_19368_amd.build.build()

Objects go to paper_2607_19368_amd/_build/, the library to
paper_2607_19368_amd/libslh.so (in-tree, next to the Python binding).
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OUT = os.path.join(PKG, "libslh.so")
OBJ = os.path.join(PKG, "_build")

SOURCES = [
    "slh_api.cpp",
    "k_prep.hip",
    "k_group.hip",
    "k_featmap.hip",
    "k_lanczos.hip",
    "k_lzres.hip",
    "k_eig.hip",
    "k_local.hip",
    "k_norm.hip",
    "k_diag.hip",
    "k_hash.hip",
    "k_merge.hip",
    "k_route.hip",
    "k_peak.hip",
    "slh_noalloc.hip",
]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 instructions are kept out of all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-pass-failed",
    "-Wshadow", "-Werror=shadow",       # a name hidden by another has cost a code path here
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(src):
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    jobs = min(len(SOURCES), int(os.environ.get("MAX_JOBS", "8")))
    with ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, OUT)
    if verbose:
        print(f"built {OUT}")
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
