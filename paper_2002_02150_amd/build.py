"""Builds the HIP library libfcas.so (gfx950) in-tree with hipcc.

    python -m paper_2002_02150_amd.build      (or python paper_2002_02150_amd/build.py)
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libfcas.so")
BUILD = os.path.join(HERE, "_build")
SOURCES = ["eval_f32.hip", "eval_f64.hip", "fcas_api.cpp", "setup.hip", "grad.hip", "pso.hip", "inject.hip", "tail.hip"]
# pass 1, one object per precision and detector count (compiled in parallel)
PASS1 = [("eval_pass1.hip", real, dt) for dt in range(8, 0, -1) for real in ("float", "double")]
ARCH = os.environ.get("FCAS_OFFLOAD_ARCH", "gfx950")


def hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def common_flags():
    return ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
            # no packed FP32 instructions anywhere in the device code
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            # multiply-adds are fused only within one source expression, so every
            # inlined copy of a tile function rounds the same way (bitwise-repeatable
            # results whatever work-group or schedule evaluates a point)
            "-ffp-contract=on",
            "-Wall", "-Wno-unused-function", "-Wno-unused-variable", "-Wno-unused-value", "-Wno-unused-result"]


def compile_one(unit):
    """unit: a source file, or (source file, FCAS_REAL, FCAS_DT)."""
    src, defs, suffix = unit, [], ""
    if isinstance(unit, tuple):
        src, real, dt = unit
        defs, suffix = [f"-DFCAS_REAL={real}", f"-DFCAS_DT={dt}"], f"_{real}_{dt}"
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + suffix + ".o")
    lang = ["-x", "hip"] if src.endswith(".cpp") else []
    cmd = [hipcc()] + common_flags() + defs + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose=True):
    os.makedirs(BUILD, exist_ok=True)
    units = SOURCES[:2] + PASS1 + SOURCES[2:]   # the longest first
    with ThreadPoolExecutor(max_workers=min(len(units), os.cpu_count() or 4)) as ex:
        objs = list(ex.map(compile_one, units))
    tmp = OUT + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, OUT)
    if verbose:
        print(f"built {OUT}")
    return OUT


if __name__ == "__main__":
    try:
        build()
    except RuntimeError as exc:
        print(exc, file=sys.stderr)
        sys.exit(1)
