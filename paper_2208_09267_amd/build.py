"""Build the gfx950 HIP library ``libvanse.so`` in-tree with hipcc.

Usage: ``python -m paper_2208_09267_amd.build`` (or ``build()`` from Python).
"""
from __future__ import annotations

import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libvanse.so")
SOURCES = ["kernels.hip", "march.hip", "box.hip", "api.hip"]
ARCH = "gfx950"

# Packed FP32 instructions are disabled on purpose: every kernel is compiled
# without them, so hipcc emits scalar-per-lane FP32 arithmetic only.
HIP_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH,
    # contract a*b+c only within one source expression, so a device function
    # compiles to the same arithmetic in every kernel that inlines it
    "-ffp-contract=on",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


def build(verbose: bool = False, extra_flags=None) -> str:
    """Compile every HIP source into ``paper_2208_09267_amd/libvanse.so``."""
    objs = []
    cc = hipcc()
    flags = HIP_FLAGS + list(extra_flags or [])
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    running = []  # the sources compile side by side
    for src in SOURCES:
        obj = os.path.join(bdir, src + ".o")
        cmd = [cc] + flags + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        running.append((subprocess.Popen(cmd), cmd))
        objs.append(obj)
    failed = [(p.returncode, cmd) for p, cmd in running if p.wait()]
    if failed:
        raise subprocess.CalledProcessError(*failed[0])
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [cc, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
