"""Decisions that hang on the last bit of a pose: a sphere's centre deep in a
cuboid with two faces equally near, where the gradient is one face's normal or
the other's.  A batch whose layout the autotuner chooses decides them as the
wave-per-link layout does, whichever layout runs."""
import os

import numpy as np
import pytest
import torch

from paper_2310_17274_amd import workloads as wl
from tests.test_parity_gpu import Case, _dev

pytestmark = pytest.mark.gpu

# collision terms alone: a few 1e4 per entry, each the sum of some 20 terms of
# at most w (5000) times a lever below 2 m, every term with a handful of
# roundings of 6e-8: below 0.1.  A normal that points along the other face moves
# an entry by w times the lever of that sphere, mostly hundreds.
ALONE = dict(a0=0.0, a1=0.0, a6=0.0, a8=0.0, a9=0.0)
TOL = 1.0


def _centres(robot, q):
    """Sphere centres [rows, M, 3] in fp64."""
    out = np.zeros((len(q), robot.n_spheres, 3))
    F = np.asarray(robot.fixed_tf, np.float64).reshape(-1, 3, 4)
    for i, row in enumerate(np.asarray(q, np.float64)):
        pose = []
        for l in range(robot.n_links):
            c, s = np.cos(row[l]), np.sin(row[l])
            A = np.eye(4)
            A[:3] = F[l]
            A = A @ np.array([[c, -s, 0, 0], [s, c, 0, 0], [0, 0, 1, 0], [0, 0, 0, 1.0]])
            pose.append(A if robot.parent[l] < 0 else pose[robot.parent[l]] @ A)
        for m, l in enumerate(robot.sphere_link):
            out[i, m] = pose[l][:3, :3] @ np.asarray(robot.sphere[m][:3], np.float64) + pose[l][:3, 3]
    return out


def _tie_case(robot, seeds, horizon, n_box, swept):
    """n_box cubes, each around one sphere of one row so that its centre lies
    on a diagonal of two axes, as near to one face as to the other."""
    rng = np.random.default_rng(31)
    robot = wl.robot_f32(robot)
    batch = wl.to_f32(wl.make_batch(robot, 32, [seeds], [horizon], [0], noise=0.02))
    q = np.asarray(batch.x0, np.float32).reshape(-1, robot.dof)
    c = _centres(robot, q)
    pose, dims = np.zeros((n_box, 7)), np.full((n_box, 3), 0.1)
    for i in range(n_box):
        off = np.zeros(3)
        off[rng.permutation(3)[:2]] = rng.choice([-1, 1], 2) * 0.03
        pose[i, :3] = c[rng.integers(len(c)), rng.integers(c.shape[1])] + off
        pose[i, 3] = 1.0
    worlds = wl.Worlds(np.array([0, n_box], np.int32), pose, dims)
    return Case(robot, worlds, batch, params=dict(ALONE, swept=swept))


def _grads(case, K):
    alpha = [0.5] * K
    d = torch.zeros_like(case.x)
    o = case.ctx.mg_linesearch_eval(case.b, case.q_start, case.goal, case.x, d, alpha)
    torch.cuda.synchronize()
    return o[2].cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("horizon,swept", [(1, 0), (6, 0), (1, 1), (6, 1)])
def test_tuned_two_arms_decide_as_wave_per_link(horizon, swept):
    case = _tie_case(wl.make_two_arm(seed=0, n_spheres=120), 24, horizon, 300, swept)
    case.b.mg_batch_set_layout(1, 1)
    want = _grads(case, 4)
    assert np.abs(want).max() > 1e4
    case.b.mg_batch_set_layout(-1, 0)
    case.ctx.mg_autotune(case.b, case.q_start, case.goal, case.x, torch.zeros_like(case.x), [0.5, 0.5], launches=2)
    # the tuned launch, and lane per link (a count that was not tuned)
    assert np.abs(_grads(case, 2) - want[:2]).max() < TOL
    assert np.abs(_grads(case, 4) - want).max() < TOL


@pytest.mark.parametrize("arms", [1, 2])
def test_swept_particles_cost_as_wave_per_link(arms):
    """Costs of 64 traced particles in the layout of their own choice: rounding
    alone (1e-6 of the cost) apart from wave per link's."""
    robot = wl.make_arm(seed=0, n_spheres=52) if arms == 1 else wl.make_two_arm(seed=0, n_spheres=60)
    case = Case(robot, wl.make_worlds(21, [60]), wl.make_batch(robot, 22, [6], [8], [0], noise=0.1),
                params=dict(swept=1))
    case.b.mg_batch_reserve_particles(64)
    costs = []
    for layout in (-1, 1):
        case.b.mg_batch_set_layout(layout, 0)
        x, var = case.x.clone(), torch.full_like(case.x, 0.01)
        o = case.ctx.mg_particles_seeded(case.b, case.q_start, case.goal, x, var, 64, 1, 5, costs=True)
        torch.cuda.synchronize()
        costs.append((o[-1] if isinstance(o, (tuple, list)) else o).cpu().numpy().astype(np.float64))
    assert np.allclose(costs[0], costs[1], rtol=1e-5, atol=0.0)


@pytest.mark.parametrize("copies", [1, 2, 4])
def test_two_arms_trace_alike_with_every_number_of_copies(copies):
    """The trace queue over five tiles of cuboids (an untuned number of
    candidates on a tuned batch)."""
    case = _tie_case(wl.make_two_arm(seed=0, n_spheres=120), 24, 6, 300, 1)
    case.b.mg_batch_set_layout(1, 1)
    want = _grads(case, 4)
    case.ctx.mg_autotune(case.b, case.q_start, case.goal, case.x, torch.zeros_like(case.x), [0.5, 0.5], launches=1)
    old = os.environ.get("MG_CUBOID_SLICES")
    os.environ["MG_CUBOID_SLICES"] = str(copies)
    try:
        got = _grads(case, 4)
    finally:
        os.environ.pop("MG_CUBOID_SLICES")
        if old is not None:
            os.environ["MG_CUBOID_SLICES"] = old
    assert np.abs(got - want).max() < TOL
