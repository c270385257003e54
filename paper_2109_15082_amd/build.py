"""Builds libmrem.so (HIP, gfx950) in-tree: python -m paper_2109_15082_amd.build"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libmrem.so")
OBJ_DIR = os.path.join(HERE, "_build")
SOURCES = ["mrem_api.hip", "mrem_elem.hip", "mrem_gemm.hip", "mrem_attn.hip", "mrem_attn_mfma.hip"]
# the products' kernels take longest to compile: one unit for each operand form of mrem_gemm.hip, and the rest of it
PARTS = {"mrem_gemm.hip": [0, 1, 2, 3, 4]}
FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    cc = hipcc()

    def compile_one(unit) -> str:
        src, part = unit
        obj = os.path.join(OBJ_DIR, src.replace(".hip", f"{'' if part is None else part}.o"))
        cmd = [cc, *FLAGS, *([] if part is None else [f"-DMREM_GEMM_PART={part}"]), "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
        if verbose and r.stderr.strip():
            # the host pass does not know the packed-fp32 target feature and says so: harmless
            lines = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip()]
            if lines:
                print("\n".join(lines), file=sys.stderr)
        return obj

    units = sorted(((s, p) for s in SOURCES for p in PARTS.get(s, [None])), key=lambda u: u[0] not in PARTS)  # the longest first
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        objs = list(ex.map(compile_one, units))
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", OUT]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    if verbose:
        print(f"built {OUT}")
    return OUT


if __name__ == "__main__":
    build()
