"""Seeds' sums made by the evaluation launch, whose rows meet between
workgroups: many launches back to back on alternating inputs, so that a row
read before its workgroup's store, or from a cache, would be the other
input's and change the sum."""
import pytest
import torch

from paper_2310_17274_amd import workloads as wl
from tests.test_parity_gpu import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seeds,horizon,K", [(32, 32, 8), (700, 33, 1), (3, 64, 16), (90, 7, 4)])
def test_alternating_inputs(seeds, horizon, K):
    """At most 24576 evaluations (more take a launch of their own): every copy
    count, seeds that workgroups share and workgroups that share a seed."""
    assert seeds * horizon * K <= 24576
    robot = wl.make_arm(seed=0, n_spheres=20)
    case = Case(robot, wl.make_worlds(31, [30]), wl.make_batch(robot, 32, [seeds], [horizon], [0], noise=0.1))
    xs = [case.x, (0.9 * case.x).contiguous()]
    d = torch.full_like(case.x, 0.01)
    alpha = [(k + 1) / K for k in range(K)]
    call = lambda i: case.ctx.mg_linesearch_eval(case.b, case.q_start, case.goal, xs[i], d, alpha, grad=False)
    want = []
    for i in range(2):
        want.append([t.clone() for t in call(i) if t is not None])
        torch.cuda.synchronize()
    assert not torch.equal(want[0][0], want[1][0])
    off = torch.zeros((), dtype=torch.int64, device="cuda")
    for n in range(400):
        for g, w in zip([t for t in call(n % 2) if t is not None], want[n % 2]):
            off += (g != w).sum()
    assert int(off) == 0
