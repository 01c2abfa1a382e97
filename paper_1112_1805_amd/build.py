"""Build script of the HIP library (gfx950).  `python -m paper_1112_1805_amd.build`."""
from __future__ import annotations

import concurrent.futures
import glob
import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libshearseg.so")
ARCH = os.environ.get("SHEARSEG_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = True) -> str:
    """Compiles every csrc/*.hip (in parallel, one kernel group each) and links the library."""
    flags = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
             # packed FP32 instructions stay off (generated code uses scalar FP32 ops)
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    # the slowest units first, so that they do not start last
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")), key=lambda f: ("mixed" not in f, f))
    tmp = OUT + ".tmp"
    with tempfile.TemporaryDirectory() as obj:
        def run(cmd):
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)

        def compile_one(src):
            o = os.path.join(obj, os.path.basename(src) + ".o")
            run([hipcc(), *flags, "-c", "-o", o, src])
            return o

        with concurrent.futures.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            objs = list(pool.map(compile_one, srcs))
        run([hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
