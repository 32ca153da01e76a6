"""Build libsimnet.so (and the peak probes, libsimnet_peaks.so) in-tree
with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsimnet.so")
SOURCES = ["kernels.hip", "split.hip", "train.hip", "abi.hip"]
PEAKS_LIB = os.path.join(HERE, "libsimnet_peaks.so")
PEAKS_SOURCES = ["peaks.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions stay off (hipcc emits them from plain float code)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fvisibility=hidden", "-Wall", "-Wno-unused-result",
]


def build(verbose: bool = False) -> str:
    _build(LIB, SOURCES, verbose)
    _build(PEAKS_LIB, PEAKS_SOURCES, verbose)
    return LIB


def _build(lib: str, sources, verbose: bool) -> None:
    """One object per source (compiled side by side), then one link."""
    tmp = lib + ".tmp"

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        proc = subprocess.run(cmd, capture_output=True, text=True)
        msgs = "\n".join(l for l in (proc.stdout + proc.stderr).splitlines()
                         if "packed-fp32-ops" not in l)
        if proc.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + msgs)
        if verbose and msgs.strip():
            print(msgs, file=sys.stderr)

    with tempfile.TemporaryDirectory() as objs, ThreadPoolExecutor(len(sources)) as pool:
        objects = [os.path.join(objs, s + ".o") for s in sources]
        list(pool.map(run, [[HIPCC, *FLAGS, "-I", os.path.join(HERE, "..", "include"), "-c",
                             os.path.join(CSRC, s), "-o", o] for s, o in zip(sources, objects)]))
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objects])
    os.replace(tmp, lib)


if __name__ == "__main__":
    print(build(verbose=True))
