"""Build the gfx950 library libpne.so from csrc/*.hip with hipcc (in-tree).

Usage: python -m paper_2603_16644_amd.build  (or call build()).
Every HIP source is compiled with -O3 for gfx950 only; packed-FP32 VALU
instructions are disabled.  The build fails where a kernel spills vector
registers: a reload from scratch memory waits for every load in flight, which
the kernels' pipelines are built around, and a version of the Cholesky step
whose MFMA operands were spilled once returned wrong values (the cause was
not found).
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libpne.so")
BUILD_DIR = os.path.join(HERE, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Wno-unused-function", "-Wno-unused-variable",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Rpass-analysis=kernel-resource-usage"]


def spills(report: str) -> list[tuple[str, int]]:
    """(kernel, spilled vector registers) of every kernel that has some, from
    the compiler's kernel-resource-usage remarks."""
    found, name = [], ""
    for key, value in re.findall(r"remark: .*?(Function Name|VGPRs Spill): (\S+)", report):
        if key == "Function Name":
            name = value
        elif int(value):
            found.append((name, int(value)))
    return found


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, "-I", os.path.join(HERE, "..", "include"), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    report = r.stderr or ""
    if r.returncode != 0:
        err = "\n".join(l for l in report.splitlines() if "packed-fp32-ops" not in l and "remark:" not in l)
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    bad = spills(report)
    if bad:
        os.remove(obj)
        raise RuntimeError(f"{src}: spilled vector registers: " + ", ".join(f"{k} ({n})" for k, n in bad))
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    jobs = min(len(srcs), int(os.environ.get("MAX_JOBS", os.cpu_count() or 4)))
    with cf.ThreadPoolExecutor(max_workers=max(1, jobs)) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
