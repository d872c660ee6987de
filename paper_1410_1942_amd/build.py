"""Build the HIP library (gfx950) in place: paper_1410_1942_amd/libpcgmi.so."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libpcgmi.so")
SOURCES = [os.path.join(CSRC, f) for f in ("kernels.hip", "resident.hip", "engine.cpp")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC",
    "--offload-arch=gfx950",
    # no packed FP32 instructions anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


def build(verbose: bool = False, extra=None) -> str:
    """Compile the sources side by side, then link them."""
    with tempfile.TemporaryDirectory(prefix="pcgmi_") as tmp:
        objs, procs = [], []
        for src in SOURCES:
            obj = os.path.join(tmp, os.path.basename(src) + ".o")
            cmd = [HIPCC, *FLAGS, *(extra or []), "-I", INCLUDE, "-I", CSRC,
                   "-c", "-x", "hip", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            objs.append(obj)
            procs.append((cmd, subprocess.Popen(cmd)))
        codes = [(cmd, q.wait()) for cmd, q in procs]
        for cmd, code in codes:
            if code:
                raise subprocess.CalledProcessError(code, cmd)
        # no undefined symbols: a lost kernel file fails here, not at run time
        subprocess.run([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-Wl,-z,defs", *objs,
                        "-o", LIB + ".tmp"], check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
    print(LIB)
