"""Builds libhvpic.so (HIP, gfx950) in-tree with hipcc.

The sources under csrc/ are compiled side by side and linked into one shared
library exporting the C-ABI of include/hvpic.h.  Packed FP32 instructions are disabled for the device code.
"""
from __future__ import annotations

import concurrent.futures
import os
import pathlib
import subprocess
import tempfile

PKG = pathlib.Path(__file__).resolve().parent
ROOT = PKG.parent
SOURCES = ["particles.hip", "sort.hip", "fields.hip", "fields_ext.hip", "open.hip", "surrogate.hip",
           "ensemble.hip", "abi.hip"]
LIB = PKG / "libhvpic.so"


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return str(pathlib.Path(rocm) / "bin" / "hipcc")


def build(verbose: bool = False, extra: list[str] | None = None) -> pathlib.Path:
    tmp = PKG / "libhvpic.so.tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
           f"-I{ROOT / 'include'}", f"-I{PKG / 'csrc'}", *(extra or [])]
    if verbose:
        print(" ".join(cmd))
    with tempfile.TemporaryDirectory() as d:
        # the sources side by side, the longest first
        objs = [pathlib.Path(d) / (s + ".o") for s in SOURCES]
        with concurrent.futures.ThreadPoolExecutor(min(len(SOURCES), os.cpu_count() or 1)) as pool:
            list(pool.map(lambda s, o: subprocess.run([*cmd, "-c", str(PKG / "csrc" / s), "-o", str(o)], check=True),
                          SOURCES, objs))
        subprocess.run([hipcc(), "--offload-arch=gfx950", "-shared", *map(str, objs), "-o", str(tmp)], check=True)
    tmp.replace(LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
