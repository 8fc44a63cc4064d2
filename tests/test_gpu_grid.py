"""The candidate grids built on the device against their reference construction on the
host, and the cell classes behind the inside test (Sec. 7.1: closest points and inside
tests of polygons and triangle meshes)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2201_13240_amd import workloads as WL
from tests.gpu_common import dev, torch_cuda

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2201_13240_amd", "csrc")
ONE = WL.field_const(1.0)
ZERO = WL.field_const(0.0)


@pytest.fixture(scope="module")
def W():
    torch_cuda()
    from paper_2201_13240_amd import wos
    wos.lib()
    return wos


@pytest.fixture(scope="module")
def reference(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("grid_total")
    exe = str(d / "grid_total")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread", f"-I{CSRC}",
                           os.path.join(HERE, "host", "grid_total.cpp"), os.path.join(CSRC, "bvh.cpp"), "-o", exe])

    def run(kind, arr):
        path = str(d / "prims.bin")
        np.ascontiguousarray(arr, np.float64).tofile(path)
        out = subprocess.run([exe, kind, path], capture_output=True, text=True, check=True).stdout.split()
        return {out[i]: int(out[i + 1]) for i in range(0, len(out), 2)}
    return run


def _problem(dim, g):
    return WL.make_problem(dim, g, ONE, ZERO, ONE, ZERO, ONE)


# 3: the smallest; 63, 65: around 4096 cells; 256; 4096: truncated lists deep inside
@pytest.mark.parametrize("edges", [3, 63, 65, 256, 4096])
def test_polygon_lists_are_the_references(W, reference, edges):
    g = WL.star_polygon(np.random.default_rng(edges), edges)
    V = g["vertices"]
    ref = reference("seg", np.c_[V, np.roll(V, -1, axis=0)])
    got = W.Problem(_problem(2, g)).grid_info()
    assert (got["nx"], got["ny"], got["candidates"]) == (ref["nx"], ref["ny"], ref["candidates"])
    assert (ref["truncated"] > 0) == (edges == 4096)


@pytest.mark.parametrize("subdiv", [0, 2, 4])
def test_mesh_lists_are_the_references(W, reference, subdiv):
    g = WL.icosphere(np.random.default_rng(subdiv), subdiv, 0.1)
    tris = np.zeros((len(g["triangles"]), 12))
    tris[:, :9] = g["vertices"][g["triangles"]].reshape(-1, 9)
    ref = reference("tri", tris)
    got = W.Problem(_problem(3, g)).grid_info()
    assert tuple(got[k] for k in ("nx", "ny", "nz", "candidates")) == tuple(
        ref[k] for k in ("nx", "ny", "nz", "candidates"))


def _winding(V, T, p):
    a, b, c = (V[T[:, k]][None] - p[:, None] for k in range(3))
    la, lb, lc = (np.linalg.norm(q, axis=2) for q in (a, b, c))
    num = (a * np.cross(b, c)).sum(2)
    den = la * lb * lc + (a * b).sum(2) * lc + (a * c).sum(2) * lb + (b * c).sum(2) * la
    return 2 * np.arctan2(num, den).sum(1)


@pytest.mark.parametrize("shape", ["sphere", "shells", "hole", "flipped"])
def test_mesh_inside(W, shape):
    """Points around a closed sphere, a sphere with a hollow core and a separate small one,
    a sphere with a missing triangle (no cell classes: every point goes through the winding
    number) and one turned inside out, against the winding number in numpy."""
    rng = np.random.default_rng(4)
    V, T = WL._icosphere_unit(2)
    V = V * (1.0 + rng.uniform(-0.1, 0.1, V.shape[0]))[:, None]
    if shape == "shells":
        n = len(V)
        V = np.concatenate([V, 0.4 * V, 0.3 * V + [2.0, 0.0, 0.0]])
        T = np.concatenate([T, T[:, ::-1] + n, T + 2 * n])
    elif shape == "hole":
        T = T[1:]
    elif shape == "flipped":
        T = T[:, ::-1]
    g = WL.geom_trimesh(V, T)
    p = rng.uniform(V.min(0) - 0.3, V.max(0) + 0.3, (3000, 3))
    d = rng.normal(size=(500, 3))
    p = np.concatenate([p, d / np.linalg.norm(d, axis=1, keepdims=True) * rng.uniform(0.85, 1.15, (500, 1))])
    w = _winding(V, T, p)
    keep = np.abs(np.abs(w) - 2 * np.pi) > 1e-6
    p = np.concatenate([p[keep], [[np.nan, 0, 0], [1e30, 0, 0]]])
    want = np.concatenate([np.abs(w[keep]) > 2 * np.pi, [False, False]])
    got = W.classify(W.Problem(_problem(3, g)), dev(p)).cpu().numpy().astype(bool)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 5000])
def test_polygon_inside(W, n):
    """Points in the bounding box and along the edges of a star polygon with a pocket, at
    counts around the block size, against the crossing count in numpy."""
    rng = np.random.default_rng(n)
    V = WL.star_polygon(np.random.default_rng(9), 301, 8, 0.6)["vertices"]
    e = rng.integers(0, len(V), n)
    t = rng.uniform(0, 1, (n, 1))
    near = (1 - t) * V[e] + t * np.roll(V, -1, axis=0)[e] + rng.normal(scale=1e-3, size=(n, 2))
    p = np.where(rng.uniform(size=(n, 1)) < 0.5, near, rng.uniform(-1.8, 1.8, (n, 2)))
    g = WL.geom_polygon(V)
    want = WL.inside_mask(g, p)
    got = W.classify(W.Problem(_problem(2, g)), dev(p)).cpu().numpy().astype(bool)
    assert np.array_equal(got, want)
