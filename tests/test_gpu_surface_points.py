"""Inside tests of points on the surface of a mesh with flat faces (Sec. 7.1: generalized
winding number), where the angles add up to the threshold and rounding decides: the answers
are those of the sum in the primitives' order, one point per thread, which the library gave
from its first inside test on. Recorded on MI355X."""
import numpy as np
import pytest

from paper_2201_13240_amd import workloads as WL
from tests.gpu_common import dev, torch_cuda
from tests.test_gpu_triangles import _cube

pytestmark = pytest.mark.gpu

# k: (points inside, flags of the 386 lattice points on the surface, packed)
FLAGS = {
    1: (167, "001c0643e070200000000005547e0011515f0017757f001515770dbf757f1dbd797f1c057c3e000f8fa7f3b9fcfe3e0000"),
    2: (145, "001d064a82a1b86408000e07c43a111d157f3bb727772431e05d0087052f041191551384b736000a8ee23048a8aa260000"),
    4: (107, "0028800aa0228000820026a0e22900020000150ccc2a0d37dc7f200406200415dc7a00a2222a00030282a3f8a0f4210000"),
}


@pytest.fixture(scope="module")
def W():
    torch_cuda()
    from paper_2201_13240_amd import wos
    wos.lib()
    return wos


@pytest.mark.parametrize("k", sorted(FLAGS))
def test_points_on_a_cube(W, k):
    t = np.arange(-4, 5) / 4.0
    p = np.stack(np.meshgrid(t, t, t, indexing="ij"), -1).reshape(-1, 3)
    p = p[np.abs(p).max(1) == 1.0]
    one = WL.field_const(1.0)
    h = W.Problem(WL.make_problem(3, WL.geom_trimesh(*_cube(k)), one, WL.field_const(0.0), one, WL.field_const(0.0),
                                  WL.field_manufactured("expcos")))
    P = dev(p)
    got = W.classify(h, P).cpu().numpy()
    assert (int(got.sum()), np.packbits(got.astype(np.uint8)).tobytes().hex()) == FLAGS[k]
    # a solve takes the same points for outside ones, and ends the walks of the others at once
    acc = W.Accumulators(len(p))
    W.solve([(h, P, acc, 0)], W.options(walks=4, seed=1))
    assert np.array_equal(np.isnan(acc.sum.cpu().numpy()), got == 0)
    assert int(acc.counters[0]) == len(p) - FLAGS[k][0]
    np.testing.assert_array_equal(acc.n_steps.cpu().numpy(), np.where(got == 1, 4, 0))
