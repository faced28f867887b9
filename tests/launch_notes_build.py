"""Builds tests/launch_notes.cpp: the host side of libfp8lm on a HIP runtime that only takes notes of launches."""
from __future__ import annotations

import os
import subprocess

from paper_2310_18313_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "launch_notes.cpp")
LIB = os.path.join(HERE, "_build", "liblaunch_notes.so")


def build(force: bool = False) -> str:
    deps = [SRC, *B.DEPS]
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in deps):
        return LIB
    os.makedirs(os.path.dirname(LIB), exist_ok=True)
    obj = LIB[:-3] + ".o"
    subprocess.check_call([
        os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-fuse-cuid=none",
        "-O1", "-std=c++17", "-ffp-contract=off", "-fPIC", "-I", os.path.join(B.ROOT, "include"), "-I", os.path.join(B.HERE, "csrc"),
        "-c", SRC, "-o", obj])
    # no device code is in it, and every symbol has to be found in it: nothing of a real runtime is linked
    subprocess.check_call(["g++", "-shared", "-o", LIB, obj, "-Wl,--defsym=__hip_fatbin=0", "-Wl,-z,defs", "-Wl,-Bsymbolic"])
    os.remove(obj)
    return LIB


if __name__ == "__main__":
    print(build(force=True))
