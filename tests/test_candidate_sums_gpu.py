"""Per-seed sums of the line-search candidates (cost, <g, d>, clearance) in
one launch, a power of two of lanes per seed: horizons at and around the
powers of two, alone and mixed in one batch, seed counts that leave the last
workgroup ragged."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("layout", [None, (0, 1), (0, 4), (3, 0)])
@pytest.mark.parametrize("horizon", [1, 32, 33])
def test_sums_made_by_the_evaluation_and_apart(horizon, layout):
    """Seed counts on both sides of the line (24576 evaluations) above which
    the sums take a launch of their own: the same bits for the seeds that both
    batches hold, call after call and in a replayed graph."""
    robot = wl.make_arm(seed=0, n_spheres=20)
    n = 24576 // horizon
    case = Case(robot, wl.make_worlds(31, [9]), wl.make_batch(robot, 32, [n + 40], [horizon], [0]), layout=layout)
    small = case.ctx.batch([n], [horizon], [0])
    if layout is not None:
        small.mg_batch_set_layout(*layout)
    run = lambda b, rows: case.ctx.mg_cost_grad(b, case.q_start, case.goal, case.x[:rows])
    c, g, mc = run(case.b, (n + 40) * horizon)
    for _ in range(2):
        c1, g1, mc1 = run(small, n * horizon)
        assert torch.equal(c1, c[:n]) and torch.equal(g1, g[:n * horizon]) and torch.equal(mc1, mc[:n])
    few = case.ctx.batch([7], [horizon], [0])
    want = [t.clone() for t in run(few, 7 * horizon)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        outs = run(few, 7 * horizon)
    for _ in range(3):
        for t in outs:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want))
        run(few, 7 * horizon)
