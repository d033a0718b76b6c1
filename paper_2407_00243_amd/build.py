"""Builds the HIP library in-tree: paper_2407_00243_amd/libtilefusion.so (gfx950 only)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtilefusion.so")
SOURCES = ["tf_kernels.hip", "tf_gemm.hip", "tf_chain.hip", "tf_gather.hip", "tf_inspector.cpp", "tf_api.cpp"]
HEADERS = ["tf_internal.h", "tf_device.h", os.path.join("..", "..", "include", "tilefusion.h")]

# packed-fp32 instructions are switched off for all device code
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-Wno-unused-command-line-argument", "-pthread"]


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    files = [os.path.join(CSRC, f) for f in SOURCES + HEADERS]
    return any(os.path.getmtime(f) > t for f in files)


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    # the sources are independent translation units: compiled side by side, then linked
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, f + ".o") for f in SOURCES]
        cmds = [[hipcc] + HIPCC_FLAGS + ["-x", "hip", "-c", os.path.join(CSRC, f), "-o", o]
                for f, o in zip(SOURCES, objs)]
        with ThreadPoolExecutor(len(cmds)) as pool:
            list(pool.map(lambda c: _run(c, verbose), cmds))
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-pthread"] + objs + ["-o", LIB], verbose)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
