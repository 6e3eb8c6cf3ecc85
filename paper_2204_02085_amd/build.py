"""Build libwfa.so for gfx950 with hipcc (in-tree, no JIT cache).

Usage: python paper_2204_02085_amd/build.py
(run as a file: importing the package itself loads the library it builds)
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libwfa.so")
SOURCES = ["kernels.hip", "api.cpp", "align.cpp", "pipeline.cpp", "server.cpp", "autotune.cpp",
           "noalloc.hip", "k_lane.hip", "k_band.hip", "k_front.hip",
           "k_adapt.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-pthread",
    # no packed-fp32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _hipcc(args) -> None:
    res = subprocess.run([HIPCC, *FLAGS, *args], capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building libwfa.so")


def build(verbose: bool = False) -> str:
    tmp = OUT + ".tmp"
    with tempfile.TemporaryDirectory() as objs:
        pairs = [(os.path.join(CSRC, s), os.path.join(objs, s + ".o")) for s in SOURCES]
        if verbose:
            print(" ".join([HIPCC, *FLAGS, *(s for s, _ in pairs)]), flush=True)
        # one compiler per source, a few at a time
        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            list(pool.map(lambda p: _hipcc(["-c", p[0], "-o", p[1]]), pairs))
        _hipcc(["-shared", "-o", tmp, *(o for _, o in pairs)])
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
