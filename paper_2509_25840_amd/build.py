"""Build the gfx950 HIP library (libchfpe.so) in-tree with hipcc: one object
per kernel family, compiled side by side, and one link."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
# longest compilations first
UNITS = ("launch_qpass_f64", "launch_pblock", "launch_pwave", "launch_pcube", "launch_hermite", "launch_qpass_f32",
         "launch_qcube", "launch_one", "chfpe")
LIB = os.path.join(HERE, "libchfpe.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions are left to nobody: the compiler must not emit them
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


def build(verbose: bool = False) -> str:
    with tempfile.TemporaryDirectory() as d:
        def compile_unit(name: str) -> str:
            obj = os.path.join(d, name + ".o")
            cmd = [HIPCC, *FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c",
                   os.path.join(CSRC, name + ".hip"), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        with ThreadPoolExecutor(min(len(UNITS), os.cpu_count() or 1)) as pool:
            objs = list(pool.map(compile_unit, UNITS))
        tmp = LIB + ".tmp"
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp], check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
