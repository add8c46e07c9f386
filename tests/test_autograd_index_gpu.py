"""MgCost's backward scales each seed's rows: with a row-to-seed index that the
first backward makes, whatever stream that runs on, and the next ones keep, also
inside a captured graph; with none where all horizons are the same."""
import numpy as np
import pytest
import torch

from paper_2310_17274_amd import workloads as wl
from paper_2310_17274_amd.binding import MgCost
from tests.test_parity_gpu import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("horizon", [[9, 1, 16], [9, 9, 9], [1, 1, 1]])
def test_backward_on_other_streams_and_captured(horizon):
    robot = wl.make_arm(seed=0, n_spheres=20)
    case = Case(robot, wl.make_worlds(31, [9, 4]), wl.make_batch(robot, 32, [5, 3, 7], horizon, [0, 1, 0]))
    assert case.b._seed_of_row is None
    _, g, _ = case.ctx.mg_cost_grad(case.b, case.q_start, case.goal, case.x)
    w = torch.linspace(0.5, 1.5, 15, device="cuda")
    rows = torch.repeat_interleave(torch.arange(15), torch.tensor(np.repeat(horizon, [5, 3, 7]))).cuda()
    want = g * w[rows].view(-1, 1)
    x = case.x.clone().requires_grad_(True)

    def grad():
        return torch.autograd.grad(MgCost.apply(x, case.ctx, case.b, case.q_start, case.goal), x, w)[0]

    torch.cuda.synchronize()
    for s in (torch.cuda.Stream(), torch.cuda.current_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            got = grad()
        s.synchronize()
        assert torch.equal(got, want)
    assert (case.b._seed_of_row is None) == (len(set(horizon)) == 1)
    # (an incoming gradient without strides, of a plain sum)
    assert torch.equal(torch.autograd.grad(MgCost.apply(x, case.ctx, case.b, case.q_start, case.goal).sum(), x)[0], g)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = grad()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        grad()
