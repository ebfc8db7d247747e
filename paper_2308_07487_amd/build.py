"""Build the sdc shared library (gfx950) in-tree.

``python -m paper_2308_07487_amd.build`` compiles every source under
``csrc/`` with hipcc, several files at a time, into
``paper_2308_07487_amd/libsdc.so``.
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libsdc.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 VALU forms stay off (see the GPU notes in the design doc)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.cpp")) +
                  glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = [ln for ln in (r.stdout + r.stderr).splitlines()
            if "packed-fp32-ops" not in ln or "error" in ln.lower()]
    if r.returncode != 0:
        sys.stderr.write("\n".join(msgs) + "\n")
        raise RuntimeError("hipcc failed building libsdc.so")
    if verbose and msgs:
        print("\n".join(msgs))


def build(verbose: bool = False) -> str:
    work = tempfile.mkdtemp(prefix="sdc_build_")
    try:
        objs = {src: os.path.join(work, os.path.basename(src) + ".o") for src in sources()}
        # the largest files first
        order = sorted(objs, key=lambda s: "fused" not in s)
        jobs = min(8, int(os.environ.get("MAX_JOBS", "8")))
        with ThreadPoolExecutor(jobs) as ex:
            list(ex.map(lambda src: _run([HIPCC, *FLAGS, "-I", os.path.join(ROOT, "include"), "-c", src, "-o", objs[src]],
                                         verbose), order))
        tmp = os.path.join(work, "libsdc.so")
        _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs.values(), "-o", tmp], verbose)
        shutil.copyfile(tmp, LIB + ".tmp")
        os.chmod(LIB + ".tmp", 0o755)
        os.replace(LIB + ".tmp", LIB)
    finally:
        shutil.rmtree(work, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
