"""Outputs of the evaluation calls laid over their inputs: read whole before
they are written."""
import ctypes as C

import pytest
import torch

from paper_2310_17274_amd import _lib
from paper_2310_17274_amd import workloads as wl
from tests.test_parity_gpu import Case

pytestmark = pytest.mark.gpu


def _eval(case, x, d, alpha, cost, gd, grad, mc, goal):
    p = lambda t: None if t is None else C.c_void_p(t.data_ptr())
    _lib.check(_lib.lib().mg_linesearch_eval(case.ctx.handle, case.b.handle, p(case.q_start), p(goal), p(x), p(d),
                                             len(alpha), (C.c_float * len(alpha))(*alpha), p(cost), p(gd), p(grad),
                                             p(mc), C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()


@pytest.mark.parametrize("horizon", [1, 16])
@pytest.mark.parametrize("layout", [(0, 1), (0, 4), (1, 1)])
def test_linesearch_eval(layout, horizon):
    robot = wl.make_arm(seed=0, n_spheres=20)
    case = Case(robot, wl.make_worlds(31, [9]), wl.make_batch(robot, 32, [300], [horizon], [0]), layout=layout)
    n = 300
    new = lambda *s: torch.empty(*s, device="cuda")
    d0 = torch.full_like(case.x, 0.05)
    for alpha in ([0.5], [0.2, 1.0]):
        K = len(alpha)
        want = [new(K, n), new(K, n), new(K, *case.x.shape), new(K, n)]
        _eval(case, case.x, d0, alpha, *want, case.goal)
        # the gradients over d (the first K rows' worth of a longer buffer), then over x
        for over in ("d", "x"):
            buf = new(K, *case.x.shape)
            buf[0] = d0 if over == "d" else case.x
            got = [new(K, n), new(K, n), buf, new(K, n)]
            _eval(case, buf[0] if over == "x" else case.x, buf[0] if over == "d" else d0, alpha, *got, case.goal)
            assert all(torch.equal(a, b) for a, b in zip(got, want)), over
        # costs and clearances over the trajectories and the directions
        x, d = torch.zeros(max(K * n, case.x.numel()), device="cuda"), torch.zeros(max(K * n, case.x.numel()), device="cuda")
        x[:case.x.numel()], d[:d0.numel()] = case.x.flatten(), d0.flatten()
        _eval(case, x, d, alpha, x, want[1].zero_(), None, d, case.goal)
        assert torch.equal(x[:K * n].view(K, n), want[0]) and torch.equal(d[:K * n].view(K, n), want[3])


@pytest.mark.parametrize("horizon", [1, 16])
def test_cost_grad(horizon):
    robot = wl.make_arm(seed=0, n_spheres=20)
    case = Case(robot, wl.make_worlds(31, [9]), wl.make_batch(robot, 32, [300], [horizon], [0]))
    cost, _, mc = case.ctx.mg_cost_grad(case.b, case.q_start, case.goal, case.x, grad=False)
    x = case.x.clone().flatten()
    p = lambda t: C.c_void_p(t.data_ptr())
    _lib.check(_lib.lib().mg_cost_grad(case.ctx.handle, case.b.handle, p(case.q_start), p(case.goal), p(x), p(x), None,
                                       p(x[1000:]), C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    assert torch.equal(x[:300], cost) and torch.equal(x[1000:1300], mc)
