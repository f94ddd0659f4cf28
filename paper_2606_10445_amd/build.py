"""Build libspense.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2606_10445_amd.build
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libspense.so")
SOURCES = ["spense_api.cpp", "spense_gemm.hip", "spense_gemm_big2.hip", "spense_gemm_mid.hip", "spense_compress.hip", "spense_quant.hip",
           "spense_index.hip", "spense_obs.hip",
           "spense_noalloc.hip"]
ARCH = "gfx950"

# -packed-fp32-ops: keep the compiler from forming packed fp32 VALU instructions.
HIP_FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang",
             "-packed-fp32-ops", "-munsafe-fp-atomics", "-Wall", "-Wno-unused-function"]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


# The compiler the kernels' explicit matrix-core wait states (xdl_fence in
# spense_gemm_device.h) were checked with: the padding it inserts across basic blocks fell
# short there, and the repeatability tests guard it (every kernel shape up to 64 tokens, the
# large-M tiles, the paired launch).  A different compiler must pass them before anything else.
CHECKED_TOOLCHAIN = ("HIP version: 7.2.26015-fc0010cf6a",
                     "AMD clang version 22.0.0git (https://github.com/RadeonOpenCompute/llvm-project roc-7.2.0 26014 "
                     "7b800a19466229b8479a78de19143dc33c3ab9b5)")


def toolchain() -> tuple[str, str]:
    """(HIP version line, clang version line) of the hipcc in use."""
    r = subprocess.run([hipcc(), "--version"], capture_output=True, text=True)
    lines = [l.strip() for l in r.stdout.splitlines()]
    hip = next((l for l in lines if l.startswith("HIP version")), "?")
    clang = next((l for l in lines if "clang version" in l), "?")
    return hip, clang


def build(verbose: bool = False) -> str:
    objdir = os.path.join(ROOT, "_build", "spense")
    os.makedirs(objdir, exist_ok=True)
    def compile_one(src: str) -> str:
        obj = os.path.join(objdir, src + ".o")
        lang = ["-x", "hip"]
        cmd = [hipcc()] + HIP_FLAGS + lang + ["-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, src),
                                               "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=4) as pool:
        objs = list(pool.map(compile_one, SOURCES))
    tmp = LIB + f".tmp{os.getpid()}"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}"] + objs + ["-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    tc = toolchain()
    print(f"toolchain: {tc[0]}; {tc[1]}", flush=True)
    if tc != CHECKED_TOOLCHAIN:
        print("WARNING: not the compiler the matrix-core wait states were checked with; run "
              "tests/test_gpu_parity.py, test_gpu_tiles128.py and test_gpu_glu.py (-k repeatable) first", flush=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
