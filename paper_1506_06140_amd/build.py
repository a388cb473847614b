"""Build libdg.so (HIP kernels for gfx950 plus the C ABI) in the package folder.

Run as ``python -m paper_1506_06140_amd.build`` or call ``build()``.  Always
recompiles.  Packed FP32 instructions are disabled for all device code.
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdg.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["dg_kernels.hip", "dg_adjoint2d.hip", "dg_line.hip", "dg_split2d.hip", "dg_march3d.hip", "dg_split3d.hip", "dg_tables.cpp"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


def build(verbose: bool = False, extra: list[str] | None = None) -> str:
    """Compile every source file (side by side) and link libdg.so."""
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as work:
        objs = [os.path.join(work, s + ".o") for s in SOURCES]
        cmds = [[HIPCC, *FLAGS, *(extra or []), "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
        if verbose:
            print("\n".join(" ".join(c) for c in cmds), flush=True)
        procs = [subprocess.Popen(c, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True) for c in cmds]
        outs = [p.communicate()[0] for p in procs]
        for p, out in zip(procs, outs):
            if p.returncode != 0 or (verbose and out):
                sys.stderr.write(out)
        if any(p.returncode for p in procs):
            raise RuntimeError("libdg build failed")
        res = subprocess.run([HIPCC, *FLAGS, "-shared", "-o", tmp, *objs], capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError("libdg link failed")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
