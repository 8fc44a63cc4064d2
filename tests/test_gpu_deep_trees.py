"""Geometries whose BVH (Sec. 7.1) is deeper than the traversal stack's column in LDS: 81,920
triangles (depth 15, 13 levels in LDS) and 20,000 edges (depth 13, 11 levels)."""
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


def _problem(kind):
    if kind == "mesh":
        return WL.make_problem(3, WL.icosphere(np.random.default_rng(3000), 6, 0.1), ONE, Z, Z, Z,
                               WL.field_manufactured("expcos"), 1e-3)
    return WL.make_problem(2, WL.star_polygon(np.random.default_rng(9), 20000), ONE, Z, Z, Z,
                           WL.field_manufactured("expcos"), 1e-3)


def _deep(dim, n, r):
    """Points around the middle, where nearly all primitives are equally far and the stack
    is fullest, the origin among them."""
    rng = np.random.default_rng(1)
    v = rng.normal(size=(n, dim))
    v *= (r * rng.random(n) ** (1.0 / dim) / np.linalg.norm(v, axis=1))[:, None]
    v[0] = 0.0
    return v


@pytest.mark.parametrize("kind,depth", [("mesh", 15), ("polygon", 13)])
def test_exact_distances(W, oracle, kind, depth):
    prob = _problem(kind)
    h = W.Problem(prob)
    assert h.bvh_info()["depth"] == depth
    p = _deep(prob["dim"], 128, 0.5)
    want, _ = oracle.distance(prob, p)
    for precision, tol in (("fp64", 4e-12), ("fp32", 8e-6)):
        d, q = (a.cpu().numpy() for a in W.eval_distance(h, dev(p), precision))
        np.testing.assert_allclose(d, want, rtol=0, atol=tol)
        np.testing.assert_allclose(np.linalg.norm(q - p, axis=1), want, rtol=0, atol=2 * tol)


@pytest.mark.parametrize("kind", ["mesh", "polygon"])
def test_harmonic_data_reproduced(W, kind):
    prob = _problem(kind)
    h = W.Problem(prob)
    p = _deep(prob["dim"], 48, 0.5)
    ex = np.exp(p[:, 0]) * np.cos(p[:, 1])
    for precision, tol in (("fp32", 2e-6), ("fp64", 1e-12)):
        r = gpu_solve(W, h, p, 2048, precision, seed=5)
        assert_parity(r["mean"], r["se"], ex, 0 * ex, f"{kind} {precision}", tol)


def test_searches_start_from_the_last_primitive(W):
    """Inner nodes per distance query of walks in the mesh: 1.058 where a search is bounded
    by the distance of the last step's triangle, 1.228 from an open bound."""
    h = W.Problem(_problem("mesh"))
    P = dev(_deep(3, 500, 0.8))
    ev = W.count_events([(h, P, W.Accumulators(len(P)), 0)], W.options(precision="fp32", walks=256, seed=6))
    assert ev["bvh_nodes"] < 1.14 * ev["steps"], ev["bvh_nodes"] / ev["steps"]
