"""Rows that are not finite among rows that are: the bounds that neighbouring
evaluations of a wave share must not spread them.  Each layout against the same
batch with the poisoned seed's rows finite."""
import numpy as np
import pytest
import torch

from paper_2310_17274_amd import workloads as wl
from tests.test_parity_gpu import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), 3.0e38])
@pytest.mark.parametrize("horizon,swept", [(1, 0), (6, 0), (1, 1), (6, 1)])
@pytest.mark.parametrize("layout", [(0, 1), (0, 2), (0, 0), (1, 1)])
def test_other_seeds_keep_their_values(layout, horizon, swept, bad):
    robot = wl.make_arm(seed=0, n_spheres=52)
    case = Case(robot, wl.make_worlds(21, [70]), wl.make_batch(robot, 22, [9], [horizon], [0], noise=0.1),
                layout=layout, params=dict(swept=swept))
    want = [t.cpu().numpy() for t in case.ctx.mg_cost_grad(case.b, case.q_start, case.goal, case.x)]
    x = case.x.clone()
    row = 4 * horizon + horizon // 2
    x[row, 2] = bad
    cost, g, mc = (t.cpu().numpy() for t in case.ctx.mg_cost_grad(case.b, case.q_start, case.goal, x))
    keep = np.arange(9) != 4
    # sums of some ten terms in another order: 1e-6 of the largest
    assert np.allclose(cost[keep], want[0][keep], rtol=1e-5, atol=0.0)
    assert np.allclose(mc[keep], want[2][keep], rtol=0.0, atol=1e-6)
    rows = np.repeat(keep, horizon)
    assert np.abs(g[rows] - want[1][rows]).max() <= 1e-5 * np.abs(want[1]).max()
    # (3e38 passes the limit by so much that the limit's cost overflows)
    assert not np.isfinite(cost[4])
