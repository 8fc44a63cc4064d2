"""The candidate lists that the device builds, entry by entry against the host reference
(Sec. 7.1): a C++ driver (tests/host/grid_records.cpp) calls the library's construction on
a BVH of its own and compares every cell's list, tail, record and band."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2201_13240_amd import workloads as WL
from tests.gpu_common import torch_cuda
from tests.test_gpu_triangles import _cube

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2201_13240_amd")
CSRC = os.path.join(PKG, "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    torch_cuda()
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("grid_records")
    exe = str(d / "grid_records")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__", f"-I{CSRC}",
                           f"-I{ROCM}/include", os.path.join(HERE, "host", "grid_records.cpp"),
                           os.path.join(CSRC, "bvh.cpp"), f"-L{PKG}", "-l:libwos.so", f"-L{ROCM}/lib", "-lamdhip64",
                           f"-Wl,-rpath,{PKG}", f"-Wl,-rpath,{ROCM}/lib", "-o", exe])

    def run(kind, arr, *more):
        path = str(d / "prims.bin")
        np.ascontiguousarray(arr, np.float64).tofile(path)
        r = subprocess.run([exe, kind, path, *more], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stderr[-2000:]
        out = r.stdout.split()
        return {out[i]: int(out[i + 1]) for i in range(0, len(out), 2)}
    return run


def _right(r, truncated):
    assert r["cells"] > 0 and (r["truncated"] > 0) == truncated, r
    assert all(r[k] == 0 for k in ("lists", "order", "tails", "inline", "floats", "bands")), r


def _segments(shape, n):
    if shape == "star":
        V = WL.star_polygon(np.random.default_rng(n), n)["vertices"]
    elif shape == "regular":    # equal distances at many cell centres
        th = 2.0 * np.pi * np.arange(n) / n
        V = np.c_[np.cos(th), np.sin(th)]
    else:                       # teeth of equal size along a square: ties, candidates of both directions
        t = np.linspace(-1.0, 1.0, n // 4 + 1)[:-1]
        w = 0.02 * (np.arange(len(t)) % 2)
        V = np.r_[np.c_[t, -1 + w], np.c_[1 - w, t], np.c_[-t, 1 - w], np.c_[-1 + w, -t]]
    return np.c_[V, np.roll(V, -1, axis=0)]


# truncated lists: where more than 32 segments are nearly equally far
@pytest.mark.parametrize("more", [[], ["deep"]], ids=["lds", "private"])
@pytest.mark.parametrize("shape,n,truncated", [("star", 3, False), ("star", 65, False), ("star", 256, False),
                                               ("star", 4096, True), ("regular", 64, True), ("teeth", 400, True)])
def test_polygon_records(driver, shape, n, truncated, more):
    _right(driver("seg", _segments(shape, n), *more), truncated)


def _triangles(shape, n):
    if shape == "ico":
        g = WL.icosphere(np.random.default_rng(n), n, 0.1)
        V, T = np.asarray(g["vertices"]), np.asarray(g["triangles"])
    elif shape == "cube":       # equal distances throughout
        V, T = _cube(n)
    else:                       # a flat set
        V = np.random.default_rng(6).uniform(-1, 1, (3 * n, 3))
        V[:, 2] = 0.0
        T = np.arange(3 * n).reshape(n, 3)
    tris = np.zeros((len(T), 12))
    tris[:, :9] = V[T].reshape(-1, 9)
    return tris


@pytest.mark.parametrize("more", [[], ["deep"]], ids=["lds", "private"])
@pytest.mark.parametrize("shape,n", [("ico", 0), ("ico", 2), ("ico", 4), ("cube", 1), ("cube", 4), ("flat", 40)])
def test_mesh_records(driver, shape, n, more):
    _right(driver("tri", _triangles(shape, n), *more), True)
