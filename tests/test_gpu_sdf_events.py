"""Event counts of SDF domains (Sec. 7.2): rows whose field a distance query evaluates, and
grid lookups."""
import numpy as np
import pytest

from paper_2201_13240_amd import workloads as WL
from tests.gpu_common import dev, torch_cuda

pytestmark = pytest.mark.gpu

ONE = WL.field_const(1.0)
Z = WL.field_const(0.0)


@pytest.fixture(scope="module")
def W():
    torch_cuda()
    from paper_2201_13240_amd import wos
    wos.lib()
    return wos


def _events(W, geometry, dim, precision):
    h = W.Problem(WL.make_problem(dim, geometry, ONE, Z, ONE, ONE, ONE), sigma_bar=2.0)
    P = dev(np.random.default_rng(3).uniform(-0.5, 0.5, (200, dim)))
    return W.count_events([(h, P, W.Accumulators(len(P)), 0)], W.options(precision=precision, walks=64, seed=2))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [5, 6, 40])
def test_only_rows_that_a_query_reads_are_counted(W, dim, n, precision):
    """A box and holes far away from it, which no cell of the box lists: one row a query
    where there are cells (six rows or more), every row of a shorter list."""
    rows = [WL.sdf_row(WL.SDF_UNION, "box", [0.0] * dim, [0.95] * dim)]
    rows += [WL.sdf_row(WL.SDF_SUBTRACT, "ball", [3.0 + 0.1 * k] * dim, [0.1]) for k in range(n - 1)]
    ev = _events(W, WL.geom_sdf(rows, [-1.0] * dim, [1.0] * dim), dim, precision)
    cells = n >= 6
    assert ev["steps"] > 200 * 64
    assert ev["prims"] == (1 if cells else n) * ev["steps"]
    assert ev["grid_cells"] == (ev["steps"] if cells else 0) and ev["bvh_nodes"] == 0


def test_scattered_scene(W):
    """33 rows, of which a query reads a few."""
    ev = _events(W, WL.csg_scatter(np.random.default_rng(6000)), 2, "fp32")
    assert ev["grid_cells"] == ev["steps"] and ev["steps"] <= ev["prims"] < 5 * ev["steps"]
