"""Closest points of triangles (paper_2201_13240_amd/csrc/triangle.h, Sec. 7.1), on CPU: a
small C++ driver (tests/host/triangle_check.cpp) compiles the device's function for the host
and holds it against brute force in FP64 and FP32, over triangles and points with small
integer coordinates in all vertex orders. There the region tests of vertices and edges
tie, which random coordinates never make them do."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2201_13240_amd", "csrc")


def test_closest_point_on_ties(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "triangle_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wno-unknown-pragmas", f"-I{CSRC}",
                           os.path.join(HERE, "host", "triangle_check.cpp"), "-o", exe])
    out = subprocess.run([exe, "20000", "1"], capture_output=True, text=True, check=True).stdout.split()
    r = {out[i]: int(out[i + 1]) for i in range(0, len(out), 2)}
    assert r["tests"] > 2_000_000 and r["ties"] > 100_000, r
    assert r["wrong64"] == 0 and r["wrong32"] == 0, r
