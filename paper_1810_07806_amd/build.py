"""Build the HIP shared library ``libwcnst.so`` for gfx950, in-tree.

The library is the C-ABI boundary declared in ``include/wcnst.h``.  Packed
FP32 instruction selection is disabled for all device code.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
SOURCES = [os.path.join(CSRC, n) for n in ("wcnst_kernels.hip", "wcnst_line.hip", "wcnst_batch.hip", "wcnst_pool.hip")]
LIB_PATH = os.path.join(PKG, "libwcnst.so")
ARCH = os.environ.get("WCNST_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"), shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    """Compile every source (side by side) and link the library."""
    flags = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-ffp-contract=off", "-fno-fast-math", "-Wall", "-Wno-unused-result",
             "-I", INCLUDE, "-I", CSRC]
    with tempfile.TemporaryDirectory(dir=PKG, prefix="_build") as tmp:
        objs = [os.path.join(tmp, os.path.basename(src) + ".o") for src in SOURCES]
        cmds = [[hipcc(), *flags, "-c", src, "-o", obj] for src, obj in zip(SOURCES, objs)]
        if verbose:
            for cmd in cmds:
                print(" ".join(cmd))
        procs = [subprocess.Popen(cmd) for cmd in cmds]
        codes = [p.wait() for p in procs]
        for cmd, rc in zip(cmds, codes):
            if rc:
                raise subprocess.CalledProcessError(rc, cmd)
        lib = os.path.join(tmp, "lib.so")
        subprocess.run([hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", lib, *objs], check=True)
        os.replace(lib, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
