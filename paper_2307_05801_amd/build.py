"""Builds the HIP library in-tree: paper_2307_05801_amd/libleap_hip.so (gfx950 only)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libleap_hip.so")
SOURCES = ["leap_geometry.cpp", "leap_host.cpp", "leap_kernels.hip", "leap_footprint_forward.hip", "leap_footprint_forward_parts.hip", "leap_footprint_back.hip",
           "leap_footprint_back_pairs.hip", "leap_footprint_back_split.hip", "leap_siddon_back_split.hip", "leap_recon.hip"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build_library(verbose: bool = False, out: str = LIB, extra_flags=()) -> str:
    """Compiles every source for gfx950, the sources side by side, and links the shared library.  Always recompiles."""
    common = [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC"]
    compile_flags = ["-c", "-x", "hip",
                     # packed FP32 instructions are kept out of the generated code on purpose
                     "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                     "-ffp-contract=fast", "-Wall", "-Wno-unused-command-line-argument",
                     "-I", os.path.join(HERE, "..", "include")] + list(extra_flags)

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        noise = "is not a recognized feature for this target"
        err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + err)
        if verbose and err.strip():
            print(err, file=sys.stderr)

    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(len(SOURCES)) as pool:
        objects = [os.path.join(tmp, s + ".o") for s in SOURCES]
        list(pool.map(run, [common + compile_flags + [os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objects)]))
        run(common + ["-shared", "-o", out] + objects)
    return out


if __name__ == "__main__":
    print(build_library(verbose=True))
