"""Jobs under a cap on the accumulation slots (wos_options.workspace_bytes): tiles shorter
than the default 256 walks, which small jobs take, need more slots and must not split a job
into more launches than the default tiles do."""
import numpy as np
import pytest

from paper_2201_13240_amd import workloads as WL
from tests.gpu_common import dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def W():
    torch_cuda()
    from paper_2201_13240_amd import wos
    wos.lib()
    return wos


# slots per point that fit: all eight of tiles of 64, four of 128, two of 256; one, for which the
# walks of a point are split into two launches
@pytest.mark.parametrize("precision", ["fp32c", "fp64"])
@pytest.mark.parametrize("fit,launches,tile", [(8, 1, 64), (7, 1, 128), (4, 1, 128), (2, 1, 256), (1, 2, 256)])
def test_short_tiles_stay_within_the_cap(W, precision, fit, launches, tile):
    g = WL.geom_box([0.0] * 3, [1.0] * 3)
    h = W.Problem(WL.make_problem(3, g, WL.field_const(1.0), WL.field_const(0.0), WL.field_const(1.0),
                                  WL.field_const(1.0), WL.field_const(0.0)), sigma_bar=1.5)
    P = dev(WL.sample_inside(np.random.default_rng(2), g, 3, 512))
    acc, ref = W.Accumulators(512), W.Accumulators(512)
    kw = dict(precision=precision, walks=512, seed=4)
    plan = W.Plan([(h, P, acc, 0)], W.options(workspace_bytes=512 * 128 * fit, **kw))
    info = plan.info()
    assert (info["launches"], info["tile_walks"]) == (launches, tile)
    plan.launch(4)
    W.solve([(h, P, ref, 0)], W.options(**kw))
    torch_cuda().cuda.synchronize()
    plan.close()
    # one rounding per point and launch
    np.testing.assert_allclose(acc.sum.cpu().numpy(), ref.sum.cpu().numpy(), rtol=4 * 2.0 ** -53, atol=0)
    assert np.array_equal(acc.n_steps.cpu().numpy(), ref.n_steps.cpu().numpy())
