"""Build libmagicdec.so (the HIP kernels and the C ABI) for gfx950, in-tree.

Each source compiles with hipcc into an object under ``_build/``; the objects
link into ``paper_2408_11049_amd/libmagicdec.so``.  Every call rebuilds.
"""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libmagicdec.so")
ARCH = "gfx950"

SOURCES = ["api.cpp", "plan.cpp", "costmodel.cpp", "attn.hip", "attn_agpr.hip", "merge.hip",
           "snapkv.hip", "step.hip", "bench.hip", "noalloc.hip"]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    path = os.path.join(rocm, "bin", "hipcc")
    return path if os.path.exists(path) else (shutil.which("hipcc") or "hipcc")


def _flags():
    return ["-std=c++17", "-O3", "-fPIC", f"--offload-arch={ARCH}", "-Wall",
            "-I", INCLUDE, "-I", CSRC,
            # No packed fp32 math in device code (v_pk_*_f32 is not emitted).
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


# Per-source flags: MFMA results in VGPRs rather than AGPRs.  snapkv.hip: the
# passes fit their register budgets either way, and the vector work that reads
# each score then needs no copy out of an AGPR.  attn.hip: measured there.
_MFMA_IN_VGPRS = ["-mllvm", "-amdgpu-mfma-vgpr-form"]
EXTRA_FLAGS = {"snapkv.hip": _MFMA_IN_VGPRS, "attn.hip": _MFMA_IN_VGPRS}


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    cmd = ([hipcc()] + _flags() + EXTRA_FLAGS.get(src, []) + lang +
           ["-c", os.path.join(CSRC, src), "-o", obj])
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False, jobs: int = 5) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
