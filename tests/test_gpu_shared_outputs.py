"""Batches whose items add into the same accumulators, or into overlapping parts of larger
ones (independent walks of one point under several problem indices, Sec. 3.1): the items
are added one after another, as if each were a call of its own."""
import numpy as np
import pytest

from paper_2201_13240_amd import workloads as WL
from tests.gpu_common import dev, torch_cuda

pytestmark = pytest.mark.gpu

NAMES = ["sum", "sum_sq", "n_walks", "n_steps", "grad_sum", "grad_sum_sq"]


@pytest.fixture(scope="module")
def W():
    torch_cuda()
    from paper_2201_13240_amd import wos
    wos.lib()
    return wos


class _View:
    """Entries `first` .. `first + n - 1` of an accumulator."""

    def __init__(self, acc, first, n):
        for k in NAMES:
            v = getattr(acc, k)
            setattr(self, k, None if v is None else v[first:first + n])
        self.counters = acc.counters


def _setup(W, gradient):
    g = WL.geom_ball([0.0, 0.0], 1.0)
    prob = WL.make_problem(2, g, WL.field_const(1.0), WL.field_const(0.0), WL.field_const(1.0), WL.field_const(1.0),
                           WL.field_manufactured("expcos"))
    h = W.Problem(prob, sigma_bar=2.0)
    pts = WL.sample_inside(np.random.default_rng(8), g, 2, 3000)
    pts[7] = [2.0, 0.0]   # outside: its sums are NaN, whichever item adds them
    return h, dev(pts), 2 if gradient else 0


def _equal(a, b, tol):
    """To `tol` times the largest sum (gradient sums of either sign cancel in part)."""
    for k in NAMES:
        if getattr(a, k) is not None:
            x, y = getattr(a, k).cpu().numpy(), getattr(b, k).cpu().numpy()
            np.testing.assert_allclose(x, y, rtol=0, atol=tol * float(np.nanmax(np.abs(y))), err_msg=k)
    np.testing.assert_array_equal(a.counters.cpu().numpy(), b.counters.cpu().numpy())


# items: (first output, points); 3 x all, overlapping halves, one point in common, one item empty
LAYOUTS = {"same": [(0, 3000)] * 3, "overlap": [(0, 2000), (1000, 2000)], "one": [(0, 257), (256, 300)],
           "empty": [(0, 600), (0, 0), (0, 600)]}


@pytest.mark.parametrize("gradient", [False, True])
@pytest.mark.parametrize("layout", sorted(LAYOUTS))
@pytest.mark.parametrize("call", ["solve", "static", "plan", "launches"])
def test_items_with_common_outputs(W, call, layout, gradient):
    h, P, gd = _setup(W, gradient)
    spans = LAYOUTS[layout]
    want, got = W.Accumulators(3000, grad_dim=gd), W.Accumulators(3000, grad_dim=gd)
    # `launches`: one slot per point and launch, 2 launches; its additions come in another order
    # (at most 5 of them, each within 2^-53 of the sum), the others' in the same
    slot = 384 if gradient else 128
    kw = dict(precision="fp32", walks=64, seed=3, tile_walks=32)
    cap = sum(n for _, n in spans) * slot if call == "launches" else 0
    for i, (f, n) in enumerate(spans):
        W.solve([(h, P[f:f + n], _View(want, f, n), i)], W.options(**kw))
    entries = [(h, P[f:f + n], _View(got, f, n), i) for i, (f, n) in enumerate(spans)]
    opt = W.options(workspace_bytes=cap, **kw)
    if call == "static":
        W.solve_static(entries, opt)
    elif call == "plan":
        plan = W.Plan(entries, opt)
        plan.launch(3)
        torch_cuda().cuda.synchronize()
        plan.close()
    else:
        W.solve(entries, opt)
    _equal(got, want, 16 * 2.0 ** -53 if call == "launches" else 0)
