"""Per-seed sums of the line-search candidates (cost, <g, d>, clearance) in
one launch, a power of two of lanes per seed: horizons at and around the
powers of two, alone and mixed in one batch, seed counts that leave the last
workgroup ragged."""
import numpy as np
import pytest

from paper_2310_17274_amd import workloads as wl
from tests.test_fullsize_gpu import _check_candidates, _direction, _oracle_candidates
from tests.test_parity_gpu import Case, _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("horizons,seeds", [([1], 300), ([2], 129), ([3], 65), ([4], 7), ([8], 33), ([9], 17),
                                            ([16], 5), ([31], 9), ([33], 5), ([64], 3), ([1, 64, 7, 32], 5)])
def test_candidate_sums(horizons, seeds):
    robot = wl.make_arm(seed=0, n_spheres=20)
    P = len(horizons)
    case = Case(robot, wl.make_worlds(31, [9]), wl.make_batch(robot, 32, [seeds] * P, horizons, [0] * P))
    alpha = [0.1, 0.6, 1.0]
    d = _direction(case, 0.1, 33)
    cost, gd, g, mc = (t.cpu().numpy() for t in case.ctx.mg_linesearch_eval(case.b, case.q_start, case.goal, case.x,
                                                                            _dev(d), alpha))
    ref_k = _oracle_candidates(case, case.batch.x0.reshape(-1, robot.dof), d, alpha)
    _check_candidates(case, cost, gd, g, mc, ref_k, d)
    c1, gd1, none, no_mc = case.ctx.mg_linesearch_eval(case.b, case.q_start, case.goal, case.x, _dev(d), alpha,
                                                       grad=False, min_clear=False)
    assert none is None and no_mc is None
    assert np.array_equal(c1.cpu().numpy(), cost) and np.array_equal(gd1.cpu().numpy(), gd)
