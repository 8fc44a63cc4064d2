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


def _sdf_rows(rng, dim, n):
    """A first shape over most of the box, then rows of every kind: runs of unions,
    intersections and subtractions, some of them repeated."""
    rows = [WL.sdf_row(WL.SDF_UNION, "box", [0.0] * dim, [0.9] * dim)]
    op = WL.SDF_SUBTRACT
    while len(rows) < n:
        if rng.uniform() < 0.3:
            op = int(rng.integers(0, 3))
        c = rng.uniform(-1.0, 1.0, dim)
        kind = rng.integers(0, 3)
        if op == WL.SDF_INTERSECT:   # keeps most of the domain
            r = WL.sdf_row(op, "ball", 0.2 * c, [rng.uniform(0.9, 1.3)])
        elif kind == 0:
            r = WL.sdf_row(op, "ball", c, [rng.uniform(0.03, 0.2)])
        elif kind == 1:
            r = WL.sdf_row(op, "box", c, rng.uniform(0.03, 0.2, dim))
        else:
            r = WL.sdf_row(op, "halfspace", c, [-rng.uniform(0.9, 1.2) * np.linalg.norm(c)])
        rows.append(rows[-1] if rng.uniform() < 0.1 and len(rows) > 1 else r)
    return np.array(rows)


def _sdf_field(rows, p):
    dim = p.shape[1]
    f = np.full(len(p), np.inf)
    for r in rows:
        c = r[2:2 + dim]
        if r[1] == 0:
            d = np.linalg.norm(p - c, axis=1) - r[5]
        elif r[1] == 1:
            q = np.abs(p - c) - r[5:5 + dim]
            d = np.where((q > 0).any(1), np.linalg.norm(np.maximum(q, 0), axis=1), q.max(1))
        else:
            d = (p @ c - r[5]) / np.linalg.norm(c)
        f = np.minimum(f, d) if r[0] == 0 else np.maximum(f, d if r[0] == 1 else -d)
    return f


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [5, 6, 7, 33, 256])
def test_sdf_cell_rows_decide_as_all_rows(W, dim, n):
    """The field from the rows a cell lists against all rows in numpy, inside, outside and
    beyond the box, for short lists (no cells), lists at the limit and long ones. FP64 to
    1e-12; FP32 to 16 units in the last place of the coordinates (about ten roundings)."""
    for seed in range(4):
        rng = np.random.default_rng([n, dim, seed])
        rows = _sdf_rows(rng, dim, n)
        p = np.concatenate([rng.uniform(-1.0, 1.0, (4000, dim)), rng.uniform(-1.5, 1.5, (500, dim))])
        h = W.Problem(_problem(dim, WL.geom_sdf(rows, [-1.0] * dim, [1.0] * dim)))
        want = -_sdf_field(rows, p)
        for precision, tol in (("fp64", 1e-12), ("fp32", 16 * 2.0 ** -24 * 2)):
            x = p if precision == "fp64" else p.astype(np.float32).astype(np.float64)
            ref = want if precision == "fp64" else -_sdf_field(rows, x)
            d, _ = W.eval_distance(h, dev(x), precision)
            np.testing.assert_allclose(d.cpu().numpy(), ref, rtol=0, atol=tol)
        got = W.classify(h, dev(p)).cpu().numpy().astype(bool)
        assert np.array_equal(got, want > 0)


def _fine_polygon(shape, n):
    th = 2.0 * np.pi * np.arange(n) / n
    if shape == "smooth":
        return WL.star_polygon(np.random.default_rng(n), n)["vertices"]
    if shape == "teeth":      # edges across the direction of the boundary
        r = np.where(np.arange(n) % 2, 1.0, 0.97)
        return np.c_[r * np.cos(th), r * np.sin(th)]
    # a strip: lists deep inside hold edges of both long sides
    m = n // 2
    x = np.linspace(-1.0, 1.0, m)
    return np.r_[np.c_[x, np.full(m, -0.15)], np.c_[x[::-1], np.full(m, 0.15)]]


# more than a sixteenth of the cells hold truncated lists, whose band most queries stop at
@pytest.mark.parametrize("shape,n", [("smooth", 2048), ("smooth", 4096), ("teeth", 3000), ("strip", 2600)])
def test_walks_in_fine_polygons_match_the_oracle(W, shape, n):
    """Estimates in polygons of many edges against the oracle's (exact distances), with bumps
    on the boundary: a step that was too long would end walks at other places of it. 128
    points, the parity criterion of all estimates."""
    from oracle import oracle as O
    from tests import parity as PR
    from tests.gpu_common import gpu_solve
    V = _fine_polygon(shape, n)
    g = WL.geom_polygon(V)
    rng = np.random.default_rng([n, 5])
    boundary = WL.field_bumps(V[rng.integers(0, n, 12)], np.full(12, 0.25), rng.uniform(-1, 1, 12))
    prob = WL.make_problem(2, g, ONE, ZERO, ZERO, ZERO, boundary)
    pts = WL.sample_inside(rng, g, 2, 128)
    ref = O.solve(prob, pts, 512, 20.0, seed=4, bvh=True)
    h = W.Problem(prob, sigma_bar=20.0)
    for precision, tol in (("fp32", 2e-6), ("fp64", 1e-12)):
        r = gpu_solve(W, h, pts, 2048, precision, seed=3)
        PR.assert_parity(r["mean"], r["se"], ref["mean"], ref["se"], f"{shape} {n} {precision}", tol)
