"""Compile the HIP sources in csrc/ for gfx950 into libbnn_hip.so beside this file (in-tree)."""
from __future__ import annotations

import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbnn_hip.so")
SOURCES = [os.path.join(CSRC, f) for f in ("bnn_api.hip", "f32_chain_bits.hip", "f32_chain_real.hip")]

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-ffp-contract=off",                                   # the fused multiply-adds are the ones written, no others
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU instructions
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources_newer_than_lib() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(HERE, "..", "include", "bnn.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def build(verbose: bool = False) -> str:
    """Always compiles (the translation units side by side).  Returns the path of the shared library."""
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.basename(src) + ".o") for src in SOURCES]
        jobs = [subprocess.Popen(["hipcc", *HIPCC_FLAGS, "-c", "-o", o, src], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
                for src, o in zip(SOURCES, objects)]
        done = [j.communicate() for j in jobs]
        err = "\n".join(ln for _, e in done for ln in e.splitlines() if "packed-fp32-ops" not in ln)
        if any(j.returncode for j in jobs):
            raise RuntimeError("hipcc failed:\n" + err)
        res = subprocess.run(["hipcc", *HIPCC_FLAGS, "-shared", "-o", LIB, *objects], capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed to link:\n" + res.stderr)
    if verbose and err.strip():
        print(err)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
