"""What can be asked of the device code without a GPU: the front end's output for gfx950, before anything is inlined, is a call
graph with the source's function names."""
import os
import re
import subprocess

import pytest

from paper_2310_18313_amd import build as B


@pytest.fixture(scope="module")
def callees(tmp_path_factory):
    """Function (mangled) -> the functions it calls."""
    out = str(tmp_path_factory.mktemp("ir") / "device.ll")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-device-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang",
                    "-disable-llvm-passes", "-emit-llvm", "-S", "-I", os.path.join(B.ROOT, "include"), "-I",
                    os.path.join(B.HERE, "csrc"), B.SRC, "-o", out], check=True, capture_output=True)
    graph, body, name = {}, None, re.compile(r'@"?([\w.$]+)"?\(')
    for line in open(out):
        if line.startswith("define"):
            body = graph.setdefault(name.search(line).group(1), set())
        elif line.startswith("}"):
            body = None
        elif body is not None and " call " in line:
            body.update(name.findall(line))
    return graph


def reachable(callees, start):
    seen, todo = set(), [start]
    while todo:
        for g in callees.get(todo.pop(), ()):
            if g not in seen:
                seen.add(g)
                todo.append(g)
    return seen


def test_scalar_epilogues_read_metadata_with_ordinary_loads(callees):
    """uniform_load reads through the constant address space, which the compiler may move past any store.  A tensor's scalar
    epilogue reads and writes the same metadata, so it has to do without."""
    def users(part):
        fs = [f for f in callees if part in f and "fp8lm" in f]
        return fs, [f for f in fs if any("12uniform_load" in g for g in reachable(callees, f))]

    begins, loading = users("5beginEi")
    assert len(begins) > 30 and len(loading) > 30           # the graph sees the loads where they belong
    finals, bad = users("8finalizeEi")
    assert len(finals) > 30
    assert not bad, bad[:3]
