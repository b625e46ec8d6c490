"""Build libdensitykv.so for gfx950 with hipcc (in-tree, next to this file).

Usage: python -m paper_2608_27922_amd.build   (or build() from Python).
Objects go to _build/ at the repository root (git-ignored)."""

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdensitykv.so")
# (source, extra flags): the Gram stages are compiled once per descriptor geometry
SOURCES = [("dkv_api.cpp", []), ("dkv_update.hip", []), ("dkv_attention.hip", []), ("dkv_sequential.hip", []),
           ("dkv_gram_f32.hip", [])] + [
    ("dkv_gram_mfma.hip", [f"-DDKV_GRAM_DESC={d}", f"-DDKV_GRAM_KV={kv}"]) for d, kv in ((64, 0), (128, 0), (128, 1), (256, 1))]
ARCH = "gfx950"

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def _hipcc():
    h = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(h):
        raise RuntimeError("hipcc not found")
    return h


def build(verbose: bool = False) -> str:
    obj_dir = os.path.join(ROOT, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(unit):
        src, extra = unit
        obj = os.path.join(obj_dir, "_".join([os.path.splitext(src)[0]] + [x.split("=")[1] for x in extra]) + ".o")
        cmd = [hipcc, "-x", "hip", *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
        if verbose and r.stderr:
            print(r.stderr, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
