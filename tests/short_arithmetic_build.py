"""Builds tests/short_arithmetic.hip, ahead of the tests (by ``__graft_entry__.build``), never inside a GPU run."""
from __future__ import annotations

import os
import subprocess

from paper_2310_18313_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "short_arithmetic.hip")
LIB = os.path.join(HERE, "_build", "libshort_arithmetic.so")


def build(force: bool = False) -> str:
    deps = [SRC, *B.DEPS]
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in deps):
        return LIB
    os.makedirs(os.path.dirname(LIB), exist_ok=True)
    # -mfma for the host half: its fused multiply-adds as instructions
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *B.HIPCC_FLAGS, "-Xarch_host", "-mfma", "-I",
                           os.path.join(B.ROOT, "include"), "-I", os.path.join(B.HERE, "csrc"), "-o", LIB, SRC])
    return LIB


if __name__ == "__main__":
    print(build(force=True))
