"""Batches in which some items ask for gradient sums (supplemental Sec. 2) and others do not:
every item gets what it gets in a batch of its own, and nothing is written for the others."""
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


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("asked", [(True, False), (False, True), (False, True, False)])
def test_each_item_as_in_a_batch_of_its_own(W, dim, precision, asked):
    g = WL.geom_ball([0.0] * dim, 1.0)
    prob = WL.make_problem(dim, g, WL.field_const(1.0), WL.field_const(0.0), WL.field_const(1.0), WL.field_const(1.0),
                           WL.field_manufactured("expcos"))
    h = W.Problem(prob, sigma_bar=2.0)
    opt = W.options(precision=precision, walks=96, seed=5)
    entries, want = [], []
    for i, gradient in enumerate(asked):
        p = WL.sample_inside(np.random.default_rng(i), g, dim, 300 + 257 * i)
        p[3] = 2.0   # outside
        entries.append((h, dev(p), W.Accumulators(len(p), grad_dim=dim if gradient else 0), i))
        # alone with gradients either way: the same walker, so the same sums bit for bit
        want.append(W.Accumulators(len(p), grad_dim=dim))
        W.solve([(h, entries[-1][1], want[-1], i)], opt)
    W.solve(entries, opt)
    for (_, _, a, i), w in zip(entries, want):
        names = ["sum", "sum_sq", "n_walks", "n_steps", "counters"]
        for k in names + (["grad_sum", "grad_sum_sq"] if asked[i] else []):
            np.testing.assert_array_equal(getattr(a, k).cpu().numpy(), getattr(w, k).cpu().numpy(), err_msg=k)
