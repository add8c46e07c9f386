"""Captured calls after mg_set_worlds: a graph of any capturable evaluation
follows the world's new cuboids and their new number, as long as the new ones
fit the allocation (larger worlds were set before)."""
import numpy as np
import pytest
import torch

from paper_2310_17274_amd import workloads as wl
from tests.test_parity_gpu import Case

pytestmark = pytest.mark.gpu


def _worlds(counts):
    """The first counts[w] cuboids of each of two worlds of ten."""
    w = wl.worlds_f32(wl.make_worlds(8, [10, 10]))
    keep = np.concatenate([np.arange(10 * i, 10 * i + n) for i, n in enumerate(counts)])
    return wl.Worlds(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), w.pose[keep], w.dims[keep])


def _call(case, what):
    ctx, b = case.ctx, case.b
    if what == "cost_grad":
        return ctx.mg_cost_grad(b, case.q_start, case.goal, case.x)
    if what == "linesearch_eval":
        return ctx.mg_linesearch_eval(b, case.q_start, case.goal, case.x, torch.full_like(case.x, 0.05), [0.3, 1.0])
    x, var = case.x.clone(), torch.full_like(case.x, 0.01)
    return ctx.mg_particles_seeded(b, case.q_start, case.goal, x, var, 32, 1, 5, costs=True)


@pytest.mark.parametrize("layout", [(-1, 0), (0, 2), (1, 2), (3, 0)])
@pytest.mark.parametrize("problems", [1, 2])
@pytest.mark.parametrize("what", ["cost_grad", "linesearch_eval", "particles"])
def test_replay_follows_the_world(what, problems, layout):
    robot = wl.make_arm(seed=0, n_spheres=52)
    batch = wl.make_batch(robot, 77, [6, 3][:problems], [8] * problems, [1, 0][:problems], noise=0.1)
    case = Case(robot, _worlds([10, 10]), batch, layout=layout)
    case.b.mg_batch_reserve_particles(32)
    case.ctx.mg_set_worlds(_worlds([3, 4]))
    _call(case, what)                                     # (allocations and code before the capture)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = _call(case, what)
    seen = []
    for counts in ([3, 4], [10, 10], [2, 7], [0, 0], [10, 9]):
        case.ctx.mg_set_worlds(_worlds(counts))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = [t.cpu().numpy() for t in out]
        want = [t.cpu().numpy() for t in _call(case, what)]
        for g, w in zip(got, want):
            assert np.array_equal(g, w)
        seen.append(want)
    # (the worlds differ for the trajectories: the last output is clearance or costs)
    assert not np.array_equal(seen[0][-1], seen[1][-1])


@pytest.mark.parametrize("layout", [(-1, 0), (1, 1), (3, 0)])
def test_solve_follows_the_world(layout):
    """mg_solve's own graph, kept over a change of the world."""
    robot = wl.make_arm(seed=0, n_spheres=52)
    batch = wl.make_batch(robot, 77, [4], [32], [1], noise=0.1)
    case = Case(robot, _worlds([10, 10]), batch, layout=layout)
    x = case.x.clone()                                    # (one buffer: the graph's key holds its address)
    for counts in ([3, 4], [10, 10], [2, 7]):
        case.ctx.mg_set_worlds(_worlds(counts))
        res = []
        for use_graph in (True, False):
            x.copy_(case.x)
            o = case.ctx.mg_solve(case.b, case.q_start, case.goal, x, 30, 4, list(wl.ALPHA_4), graph_inner=6,
                                  use_graph=use_graph)
            torch.cuda.synchronize()
            res.append([t.cpu().numpy().copy() for t in o])
        for g, w in zip(*res):
            assert np.array_equal(g, w)
