"""What decides on a batch's launch shape: mg_batch_set_layout, the autotuner,
the library's default, in any order."""
import os

import numpy as np
import pytest
import torch

from paper_2310_17274_amd import _lib
from paper_2310_17274_amd import workloads as wl
from tests.test_fullsize_gpu import _check_candidates, _direction, _oracle_candidates
from tests.test_parity_gpu import Case, _dev

pytestmark = pytest.mark.gpu


def _case(seeds=3, horizon=7, n_box=130, **kw):
    """A world crowded enough that every number of copies sums in an order of
    its own."""
    robot = wl.make_arm(seed=0, n_spheres=52)
    return Case(robot, wl.make_worlds(21, [n_box]), wl.make_batch(robot, 22, [seeds], [horizon], [0], noise=0.1), **kw)


def _eval(case, K=4):
    o = case.ctx.mg_linesearch_eval(case.b, case.q_start, case.goal, case.x, torch.full_like(case.x, 0.05),
                                    [float(a) for a in np.linspace(0.05, 1.0, K)])
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in o]


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("tuned", [False, True])
@pytest.mark.parametrize("swept", [0, 1])
def test_slices_of_the_default_layout(swept, tuned):
    """Layout -1 with a slice count is lane per link with that many copies,
    before and after an autotuning."""
    case = _case(params=dict(swept=swept))
    seen = []
    for slices in (1, 2, 4):
        if tuned:
            case.ctx.mg_autotune(case.b, case.q_start, case.goal, case.x, torch.zeros_like(case.x), [0.5, 1.0],
                                 launches=1)
        case.b.mg_batch_set_layout(-1, slices)
        got = _eval(case)
        case.b.mg_batch_set_layout(0, slices)
        assert _same(got, _eval(case))
        seen.append(got)
    assert not _same(seen[0], seen[1]) and not _same(seen[1], seen[2])


def test_refused_layout_changes_nothing():
    case = _case()
    case.b.mg_batch_set_layout(-1, 2)
    want = _eval(case)
    for bad in ((3, 2), (0, 8), (1, 5), (5, 0)):
        with pytest.raises(_lib.MgError):
            case.b.mg_batch_set_layout(*bad)
        assert _same(_eval(case), want)


def _solve(case, K, x, use_graph):
    """Six iterations, or two replays of a graph of three."""
    x.copy_(case.x)
    o = case.ctx.mg_solve(case.b, case.q_start, case.goal, x, 6, 4, [float(a) for a in np.linspace(0.1, 1.0, K)],
                          graph_inner=3, use_graph=use_graph)
    torch.cuda.synchronize()
    return [t.cpu().numpy().copy() for t in o]


def test_solve_graph_is_that_of_the_shape_asked_for():
    """A graph captured under one launch shape is not replayed under another:
    copies by the library's rule, by the environment, by the autotuner's choice
    for another number of candidates, by the caller."""
    case = _case(horizon=9)
    x = torch.empty_like(case.x)                          # (one buffer: the graph's key holds its address)
    seen = []

    def check():
        got = _solve(case, 4, x, True)
        assert _same(got, _solve(case, 4, x, False))
        seen.append(got)

    check()
    old = os.environ.get("MG_CUBOID_SLICES")
    try:
        for n in ("1", "2", "4"):
            os.environ["MG_CUBOID_SLICES"] = n
            check()
    finally:
        os.environ.pop("MG_CUBOID_SLICES")
        if old is not None:
            os.environ["MG_CUBOID_SLICES"] = old
    check()
    assert not _same(seen[1], seen[2]) and not _same(seen[2], seen[3]) and _same(seen[0], seen[4])
    choice = case.ctx.mg_autotune(case.b, case.q_start, case.goal, case.x, torch.zeros_like(case.x), [0.5, 1.0],
                                  launches=2)
    check()                                               # (not the count that was tuned)
    case.b.mg_batch_set_layout(*((0, choice) if choice in (1, 2, 4) else (1, 1)))
    check()
    for layout in ((-1, 1), (0, 4), (-1, 0), (1, 1), (1, 2), (3, 0), (2, 0)):
        case.b.mg_batch_set_layout(*layout)
        check()


def test_autotuner_times_the_default_shape():
    """A batch so small that its default is eight copies: tuned, it is the
    default's bits or another option's, never a slower shape for want of having
    timed the default (its choice is one of the numbers that the header lists)."""
    case = _case(seeds=2, horizon=3, n_box=20)
    want = _eval(case, K=2)
    choice = case.ctx.mg_autotune(case.b, case.q_start, case.goal, case.x, torch.zeros_like(case.x), [0.5, 1.0],
                                  launches=3)
    assert choice in (1, 2, 4, 8, -1, -2, -4, -8, -16, -32)
    got = _eval(case, K=2)
    for a, b in zip(got, want):
        assert np.allclose(a, b, rtol=1e-5, atol=1e-5 * np.abs(b).max())
    if choice == 8:
        assert _same(got, want)


@pytest.mark.parametrize("seeds,K", [(8, 8), (64, 8), (65, 8), (128, 4), (129, 4), (256, 8)])
def test_tuned_batches_fold_up_to_one_workgroup_a_cu(seeds, K):
    """With self-collision the tuner has wave per link alone to choose from (one
    slot group): such a batch folds its choices up to 256 workgroups of 64
    evaluations, a layout fixed by the caller at every size, two waves per
    link never."""
    robot = wl.make_arm(seed=0, n_spheres=52)
    case = Case(robot, wl.make_worlds(8, [4]), wl.make_batch(robot, 77, [seeds], [32], [0]),
                self_pairs=wl.self_pairs(robot))
    alpha = [float(a) for a in np.linspace(0.1, 1.0, K)]
    choice = case.ctx.mg_autotune(case.b, case.q_start, case.goal, case.x, torch.zeros_like(case.x), alpha, launches=1)
    assert choice < 0
    assert bool(case.ctx.mg_solve_fuses(case.b, K, 4, case.x)) == (choice != -8 and seeds * 32 * K // 64 <= 256)
    case.b.mg_batch_set_layout(1, 1)
    assert case.ctx.mg_solve_fuses(case.b, K, 4, case.x)
    case.b.mg_batch_set_layout(2, 0)
    assert not case.ctx.mg_solve_fuses(case.b, K, 4, case.x)


@pytest.mark.parametrize("horizon", [1, 2, 9])
@pytest.mark.parametrize("arms", [1, 2])
def test_tuned_traced_evaluation(arms, horizon):
    """Poses formed link by link in the lane layout (a tuned batch that traces),
    at a number of candidates that was tuned and at one that was not, against
    the FP64 reference."""
    robot = wl.make_arm(seed=0, n_spheres=23) if arms == 1 else wl.make_two_arm(seed=0, n_spheres=50)
    case = Case(robot, wl.make_worlds(21, [12]), wl.make_batch(robot, 22, [5], [horizon], [0], noise=0.1),
                params=dict(swept=1))
    d = _direction(case, 0.1, 23)
    case.ctx.mg_autotune(case.b, case.q_start, case.goal, case.x, _dev(d), [0.5, 1.0], launches=1)
    for K in (2, 4):
        alpha = [float(a) for a in np.linspace(0.05, 1.0, K)]
        cost, gd, g, mc = (t.cpu().numpy() for t in case.ctx.mg_linesearch_eval(
            case.b, case.q_start, case.goal, case.x, _dev(d), alpha))
        ref_k = _oracle_candidates(case, case.batch.x0.reshape(-1, robot.dof), d, alpha)
        _check_candidates(case, cost, gd, g, mc, ref_k, d)
