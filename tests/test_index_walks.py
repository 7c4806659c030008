"""The kernels' walks over the arcs of a row stay inside it at the largest arc
index a graph may have (tests/index_walk_main.cpp, built for the host)."""
import os
import subprocess
import tempfile

import pytest

from paper_2603_14895_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_index_walks_at_the_largest_graph():
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not installed")
    with tempfile.TemporaryDirectory() as td:
        exe = os.path.join(td, "index_walks")
        cmd = [hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-fwrapv",
               "-I", build.CSRC, os.path.join(ROOT, "tests", "index_walk_main.cpp"), "-o", exe]
        subprocess.run(cmd, check=True, capture_output=True, text=True, timeout=300)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and "index walks ok" in r.stdout, r.stdout + r.stderr
