"""Closest points of meshes with flat faces, at query points straight above their vertices
and in the planes through them (Sec. 7.1): the region tests of the triangles tie there. The
faces are cut around their centres, each centre the last vertex of all its triangles."""
import numpy as np
import pytest

from paper_2201_13240_amd import workloads as WL
from tests.gpu_common import dev, gpu_solve, torch_cuda
from tests.parity import assert_parity

pytestmark = pytest.mark.gpu

ONE = WL.field_const(1.0)
Z = WL.field_const(0.0)


@pytest.fixture(scope="module")
def W():
    torch_cuda()
    from paper_2201_13240_amd import wos
    wos.lib()
    return wos


def _cube(k):
    """[-1, 1]^3, k x k squares a face, each cut into four triangles around its centre."""
    V, T = [], []
    t = np.linspace(-1.0, 1.0, k + 1)
    for ax in range(3):
        u, v = (ax + 1) % 3, (ax + 2) % 3
        for s in (-1.0, 1.0):
            for i in range(k):
                for j in range(k):
                    q = [(t[i], t[j]), (t[i + 1], t[j]), (t[i + 1], t[j + 1]), (t[i], t[j + 1])]
                    q = q if s > 0 else q[::-1]
                    n = len(V)
                    for a, b in q + [(0.5 * (t[i] + t[i + 1]), 0.5 * (t[j] + t[j + 1]))]:
                        p = np.zeros(3)
                        p[ax], p[u], p[v] = s, a, b
                        V.append(p)
                    T += [[n + e, n + (e + 1) % 4, n + 4] for e in range(4)]
    V, inv = np.unique(np.array(V), axis=0, return_inverse=True)
    return V, inv.reshape(-1)[np.array(T)]


def _cylinder(n):
    """A prism over a regular n-gon of radius 1, height 2, its caps fans around their centres."""
    th = 2.0 * np.pi * np.arange(n) / n
    rim = np.c_[np.cos(th), np.sin(th)]
    V = np.r_[np.c_[rim, np.full(n, -1.0)], np.c_[rim, np.full(n, 1.0)], [[0, 0, -1.0], [0, 0, 1.0]]]
    T = []
    for i in range(n):
        j = (i + 1) % n
        T += [[j, i, 2 * n], [n + i, n + j, 2 * n + 1], [i, j, n + j], [i, n + j, n + i]]
    return V, np.array(T)


def _check(W, V, T, p, want, on_surface):
    h = W.Problem(WL.make_problem(3, WL.geom_trimesh(V, T), ONE, Z, ONE, Z, ONE))
    # FP32: coordinates up to 2, a dozen roundings
    for precision, tol in (("fp64", 1e-13), ("fp32", 2.0 * 12 * 2.0 ** -24)):
        x = p.astype(np.float32).astype(np.float64)
        assert np.array_equal(x, p) or precision == "fp64"
        d, q = (a.cpu().numpy() for a in W.eval_distance(h, dev(p), precision))
        np.testing.assert_allclose(d, want, rtol=0, atol=tol)
        np.testing.assert_allclose(np.linalg.norm(q - p, axis=1), want, rtol=0, atol=2 * tol)
        assert np.max(on_surface(q)) <= 2 * tol


@pytest.mark.parametrize("k", [1, 2, 4])
def test_cube_cut_around_face_centres(W, k):
    """Lattice points inside, on and outside the cube, against its distance in closed form."""
    t = np.arange(-14, 15) / 8.0
    p = np.stack(np.meshgrid(t, t, t, indexing="ij"), -1).reshape(-1, 3)
    q = np.abs(p) - 1.0
    want = np.where((q <= 0).all(1), -q.max(1), np.linalg.norm(np.maximum(q, 0.0), axis=1))
    V, T = _cube(k)
    _check(W, V, T, p, want, lambda x: np.abs(np.abs(x).max(1) - 1.0))


@pytest.mark.parametrize("n", [4, 12])
def test_cylinder_with_fan_caps(W, n):
    """Points on the axis, from end to end, and in planes through it: inside a convex body
    the distance is the smallest one to the planes of its faces."""
    z = np.arange(-31, 32) / 32.0
    r = np.arange(0, 6) / 16.0
    p = np.concatenate([np.c_[0 * z + a, 0 * z + b, z] for a in r for b in r])
    m = 2.0 * np.pi * (np.arange(n) + 0.5) / n
    side = np.cos(np.pi / n) - (p[:, :1] * np.cos(m) + p[:, 1:2] * np.sin(m)).max(1)
    want = np.minimum(1.0 - np.abs(p[:, 2]), side)
    V, T = _cylinder(n)
    _check(W, V, T, p, want, lambda x: np.zeros(1))


def test_walks_from_ties_keep_the_harmonic_solution(W):
    """u = e^x cos y in the cube, from its centre and other points whose first ball is
    decided straight above a vertex: a ball that leaves the domain would end at wrong places."""
    V, T = _cube(1)
    prob = WL.make_problem(3, WL.geom_trimesh(V, T), ONE, Z, Z, Z, WL.field_manufactured("expcos"), 1e-4)
    h = W.Problem(prob)
    c = np.arange(-3, 4) / 4.0
    p = np.concatenate([np.eye(3)[i] * a for i in range(3) for a in c[:, None, None]]).reshape(-1, 3)
    ex = np.exp(p[:, 0]) * np.cos(p[:, 1])
    for precision, tol in (("fp32", 2e-6), ("fp64", 1e-12)):
        r = gpu_solve(W, h, p, 16384, precision, seed=6)
        assert_parity(r["mean"], r["se"], ex, 0 * ex, f"cube {precision}", tol)
