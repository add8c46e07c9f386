"""Performance cases of the batched trajectory optimizer.

Each case is one call pattern of a user's program on seeded synthetic inputs:
costs with gradients at given trajectories, line-search candidates, solver
steps and short solves, the particle stage, graph-edge steering and the
planner's neighbour search, on the 7-joint arm and the two-arm tree.  `exact`
gives the same results in 64-bit arithmetic, written here from the cost's
definition in plain torch.
"""
import math

import numpy as np
import torch

from paper_2310_17274_amd import workloads as wl
from paper_2310_17274_amd.binding import Context, MgCost, default_params, mg_knn

ALPHAS = {4: wl.ALPHA_4, 8: wl.ALPHA_8}


def listed():
    arm = dict(arms=1, spheres=52, boxes=40, problems=1, swept=0)
    return [
        # the smallest call: one problem's four seeds, as a program checks or polishes one motion
        dict(arm, name="cost_grad_4x32", op="cost_grad", seeds=4, horizon=32, spheres=20, boxes=10),
        # a program's own loop over the library's solver steps on that problem (cost, then two
        # rounds of L-BFGS direction and line search)
        dict(arm, name="steps_4x32x4", op="steps", seeds=4, horizon=32, spheres=20, boxes=10, K=4, rounds=2),
        # a differentiable cost inside a torch program: forward and backward
        dict(arm, name="autograd_32x32", op="autograd", seeds=32, horizon=32),
        # candidates of one problem's line search, the optimizer's inner evaluation, layout tuned
        dict(arm, name="candidates_32x32x8", op="candidates", seeds=32, horizon=32, K=8, tuned=True),
        # the same for thousands of inverse-kinematics goals at once
        dict(arm, name="candidates_ik_4096x32x4", op="candidates", problems=4096, seeds=32, horizon=1, K=4, tuned=True),
        # a server's batch of 64 unequal problems, each in its own world of 5 to 200 cuboids
        dict(arm, name="candidates_uneven_64", op="candidates", problems=64, seeds=0, horizon=0, boxes=0, K=4,
             tuned=True),
        # two arms on one base in a dense world with continuous collision checking: the largest robot and world
        dict(arm, name="candidates_two_arm_swept", op="candidates", arms=2, spheres=120, boxes=500, seeds=128,
             horizon=48, K=4, swept=1, tuned=True),
        # the particle stage that moves the seeds before the gradient-based solve
        dict(arm, name="particles_32x32x128", op="particles", seeds=32, horizon=32, particles=128, rounds=2),
        # a short warm-started solve (graph replay), as in replanning; few enough iterations
        # that a rounding difference does not grow into another local minimum
        dict(arm, name="solve_32x32x8", op="solve", seeds=32, horizon=32, K=8, iters=12, tuned=True),
        # 16 problems with the self-collision term on
        dict(arm, name="self_collision_16x12x32", op="cost_grad", problems=16, seeds=12, horizon=32, self_pairs=True),
        # the geometric planner's batched steering: 256 edges of up to 128 steps
        dict(arm, name="steer_256x129", op="steer", edges=256, steps=128),
        # nearest nodes of a dense roadmap, every node against all
        dict(name="knn_12000", op="knn", nodes=12000, queries=12000, k=11, dof=7),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["cost_grad", "cost_grad", "steps", "autograd", "candidates", "candidates", "candidates",
                     "particles", "solve", "self", "steer", "knn"])
    if op == "knn":
        return dict(op="knn", nodes=_log(rng, 20, 12000), queries=_log(rng, 1, 12000), k=rng.randint(1, 24),
                    dof=rng.choice([7, 7, 14]))
    c = dict(arms=1, spheres=rng.randint(14, 52), boxes=_log(rng, 5, 120), problems=1, swept=0)
    if op == "steer":
        return dict(c, op="steer", edges=_log(rng, 1, 256), steps=rng.randint(16, 128))
    c.update(op=op, seeds=_log(rng, 1, 48), horizon=rng.choice([1, 8, 16, 24, 31, 32, 48]))
    if op == "self":
        return dict(c, op="cost_grad", problems=rng.randint(1, 16), seeds=rng.randint(1, 12), self_pairs=True,
                    swept=rng.choice([0, 0, 1]))
    if op in ("candidates", "cost_grad") and rng.random() < 0.3:      # two arms, continuous collision checking
        c.update(arms=2, spheres=rng.randint(28, 120), boxes=_log(rng, 20, 250), swept=rng.choice([0, 1, 1]))
    elif op in ("candidates", "cost_grad") and rng.random() < 0.4:    # several problems
        c.update(problems=_log(rng, 2, 1024), seeds=rng.randint(4, 32), horizon=rng.choice([1, 1, 8]))
    if op in ("candidates", "steps", "solve"):
        c.update(K=rng.choice([4, 8]))
    if op in ("candidates", "solve"):
        c.update(tuned=rng.random() < 0.7)
    if op == "steps":
        c.update(rounds=rng.randint(1, 2))
    if op == "solve":
        c.update(iters=rng.randint(4, 12))
    if op == "particles":
        c.update(seeds=_log(rng, 1, 32), particles=rng.choice([16, 50, 64, 100, 128]), rounds=rng.randint(1, 2))
    return c


# ---------------------------------------------------------------------------
# inputs

def _robot(case):
    if case["arms"] == 2:
        return wl.robot_f32(wl.make_two_arm(seed=0, n_spheres=case["spheres"]))
    return wl.robot_f32(wl.make_arm(seed=0, n_spheres=case["spheres"]))


def _worlds(seed, counts):
    """Oriented cuboids of the workload generator, made smaller in worlds of more than 40 so
    that a world's obstacles take the volume of 40 (a scene cut into finer pieces)."""
    w = wl.make_worlds(seed, counts, oriented=True)
    scale = np.minimum(1.0, np.cbrt(40.0 / np.maximum(1, counts)))
    w.dims = w.dims * np.repeat(scale, counts)[:, None]
    return wl.worlds_f32(w)


def _scene(case, seed):
    """Robot, worlds and the problems' layout; sizes come from the case, the
    cuboids from the seed (64 unequal problems: sizes from a fixed draw)."""
    robot = _robot(case)
    if case.get("seeds") == 0:
        r = np.random.default_rng(4)
        P = case["problems"]
        seeds, horizon = r.integers(4, 65, P), r.choice([24, 32, 48], P)
        counts, world = r.integers(5, 201, P), np.arange(P)
    else:
        P = case["problems"]
        seeds = np.full(P, case.get("seeds", 1))
        horizon = np.full(P, case.get("horizon", 1))
        counts, world = np.array([case["boxes"]]), np.zeros(P, dtype=np.int64)
    return robot, _worlds(seed, counts), seeds, horizon, world


def _unit_quat(rng, n):
    q = rng.normal(size=(n, 4))
    return q / np.linalg.norm(q, axis=1, keepdims=True)


def _depth(robot, worlds, w, q, chunk=32768):
    """How far inside the cuboids of world w the deepest sphere centre of each
    configuration q [n, D] lies (negative: outside all of them)."""
    ex = _Exact(robot, 0)
    W, out = _World(*worlds.world(int(w)), ex.dev), []
    for a in range(0, len(q), chunk):
        c = ex.fk(torch.as_tensor(q[a:a + chunk], dtype=torch.float64, device=ex.dev))[0]
        d = torch.full((len(c),), -1.0, dtype=torch.float64, device=ex.dev)
        for i in range(len(W.h)):
            p = (c - W.t[i]) @ W.R[i]
            d = torch.maximum(d, -(p.abs() - W.h[i]).amax(2).amin(1))
        out.append(d)
    return torch.cat(out).cpu().numpy()


def _least(depth, n):
    return np.argsort(np.round(depth, 6), kind="stable")[:n]


def _inputs(case, seed):
    """numpy float32 inputs as an optimizer meets them on the way, with most
    of the robot clear of the obstacles: starts that are the clearest of 32
    random configurations, goal poses (0.3 to 0.8 m away, any orientation),
    seed trajectories on noisy lines from the start to the clearest of four
    endpoints within 0.8 rad (at horizon 1, the clearest sixth of random
    configurations) and search directions."""
    robot, worlds, seeds, horizon, world = _scene(case, seed)
    rng = np.random.default_rng(1000 + seed)
    P, D = len(seeds), robot.dof
    n = P * robot.n_ee
    v = rng.normal(size=(n, 3))
    v *= (np.cbrt(rng.uniform(0.3 ** 3, 0.8 ** 3, n)) / np.linalg.norm(v, axis=1))[:, None]
    goal = np.concatenate([v, _unit_quat(rng, n)], 1).reshape(P, -1)
    S = np.repeat(np.arange(P), seeds)                     # problem of each seed
    T = horizon[S]
    q0, x = np.zeros((P, D)), []
    if (horizon == 1).all():
        q0 = rng.uniform(-1, 1, (P, D))
        pool = rng.uniform(-2.5, 2.5, (6 * len(S), D))
        x = pool[np.sort(_least(_depth(robot, worlds, 0, pool), len(S)))]
    else:
        if len(worlds.offsets) == 2:                       # one world: every problem at once
            groups = [np.arange(P)]
        else:
            groups = [np.array([p]) for p in range(P)]
        for g in groups:
            c = rng.uniform(-2, 2, (32 * len(g), D))
            dep = _depth(robot, worlds, world[g[0]], c).reshape(len(g), 32)
            q0[g] = c.reshape(len(g), 32, D)[np.arange(len(g)), np.round(dep, 6).argmin(1)]
            sg, Tg = np.repeat(g, seeds[g]), int(horizon[g[0]])
            end = q0[sg][:, None] + rng.uniform(-0.8, 0.8, (len(sg), 4, D))
            f = np.array([0.34, 0.67, 1.0])[:, None]
            probe = q0[sg][:, None, None] * (1 - f) + end[:, :, None] * f
            dep = _depth(robot, worlds, world[g[0]], probe.reshape(-1, D)).reshape(len(sg), 4, 3).max(2)
            end = end[np.arange(len(sg)), np.round(dep, 6).argmin(1)]
            f = (np.arange(1, Tg + 1) / Tg)[:, None]
            tr = q0[sg][:, None] * (1 - f) + end[:, None] * f + rng.normal(0, 0.02, (len(sg), Tg, D))
            x.append(tr.reshape(-1, D))
        x = np.concatenate(x)
    x = np.clip(x, robot.q_lo, robot.q_hi)
    d = np.clip(rng.normal(0, 0.02, x.shape), -0.06, 0.06)
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)
    return robot, worlds, seeds, horizon, world, f32(q0), f32(goal), f32(x), f32(d)


def _steer_inputs(case, seed, robot):
    rng = np.random.default_rng(2000 + seed)
    a = rng.uniform(-2, 2, (case["edges"], robot.dof))
    b = np.clip(a + rng.uniform(-1.2, 1.2, a.shape), -2.7, 2.7)
    return a.astype(np.float32), b.astype(np.float32), float(np.float32(1.25 / case["steps"]))


def _knn_inputs(case, seed):
    rng = np.random.default_rng(3000 + seed)
    nodes = rng.uniform(-2.8, 2.8, (case["nodes"], case["dof"])).astype(np.float32)
    return nodes, rng.uniform(-2.8, 2.8, (case["queries"], case["dof"])).astype(np.float32)


def prepare(case, seed):
    dev = "cuda"
    up = lambda a: torch.as_tensor(a, device=dev).contiguous()
    if case["op"] == "knn":
        nodes, queries = _knn_inputs(case, seed)
        return dict(op="knn", nodes=up(nodes), queries=up(queries), k=case["k"])
    if case["op"] == "steer":
        robot, worlds, _, _, _ = _scene(case, seed)
        ctx = Context(robot)
        ctx.mg_set_worlds(worlds)
        a, b, res = _steer_inputs(case, seed, robot)
        batch = ctx.batch([case["edges"] * (case["steps"] + 1)], [1], [0], K_max=1, m_max=0)
        return dict(op="steer", ctx=ctx, b=batch, a=up(a), to=up(b), res=res, steps=case["steps"])
    robot, worlds, seeds, horizon, world, q0, goal, x, d = _inputs(case, seed)
    ctx = Context(robot, default_params(swept=1, sweep_steps=4) if case["swept"] else None)
    ctx.mg_set_worlds(worlds)
    if case.get("self_pairs"):
        ctx.mg_set_self_collision(wl.self_pairs(robot))
    K = case.get("K", 1)
    b = ctx.batch(seeds, horizon, world, K_max=K, m_max=4 if K > 1 else 0)
    s = dict(op=case["op"], ctx=ctx, b=b, q0=up(q0), goal=up(goal), x0=up(x), d=up(d), alpha=ALPHAS.get(K, (1.0,)),
             rounds=case.get("rounds", 0), iters=case.get("iters", 0), n=case.get("particles", 0), seed=seed)
    s["x"], s["var"] = s["x0"].clone(), torch.empty_like(s["x0"])
    if case.get("tuned"):
        ctx.mg_autotune(b, s["q0"], s["goal"], s["x0"], s["d"], s["alpha"], launches=3)
    if case["op"] == "particles":
        b.mg_batch_reserve_particles(s["n"])
    if case["op"] == "autograd":
        s["w"] = up(np.random.default_rng(seed).uniform(0.5, 1.5, b.n_seeds).astype(np.float32))
        s["x"] = s["x0"].clone().requires_grad_(True)
    return s


def run(s):
    op = s["op"]
    if op == "knn":
        return mg_knn(s["nodes"], s["queries"], s["k"])
    ctx, b = s["ctx"], s["b"]
    if op == "steer":
        return ctx.mg_steer(b, s["a"], s["to"], s["res"], s["steps"])
    if op == "cost_grad":
        return ctx.mg_cost_grad(b, s["q0"], s["goal"], s["x0"])
    if op == "autograd":
        cost = MgCost.apply(s["x"], ctx, b, s["q0"], s["goal"])
        return cost.detach(), torch.autograd.grad(cost, s["x"], s["w"])[0]
    if op == "candidates":
        return ctx.mg_linesearch_eval(b, s["q0"], s["goal"], s["x0"], s["d"], s["alpha"])
    if op == "steps":
        x = s["x0"]
        c, g, mc = ctx.mg_cost_grad(b, s["q0"], s["goal"], x)
        for i in range(s["rounds"]):
            d = ctx.mg_lbfgs_step(b, 4, i == 0, x, g)
            x, c, g, chosen, mc = ctx.mg_linesearch(b, s["q0"], s["goal"], x, c, g, d, s["alpha"])
        return x, c, g, chosen, mc
    if op == "particles":
        s["x"].copy_(s["x0"])
        s["var"].fill_(0.05 ** 2)
        return ctx.mg_particles_seeded(b, s["q0"], s["goal"], s["x"], s["var"], s["n"], s["rounds"], s["seed"],
                                       costs=True)
    s["x"].copy_(s["x0"])
    return ctx.mg_solve(b, s["q0"], s["goal"], s["x"], s["iters"], 4, s["alpha"], graph_inner=4)


def work(case):
    """Bytes of the inputs and outputs once; operations of an evaluation: 170
    per link (chain and adjoint), 200 per joint, 18 per sphere (its centre),
    300 for the pose, and 20 per link and cuboid (one bounding test each:
    what a perfect cull cannot do without)."""
    op = case["op"]
    if op == "knn":
        n, m, D = case["nodes"], case["queries"], case["dof"]
        return dict(bytes=4 * (n * D + m * D + 2 * m * case["k"]), flops=3 * n * m * D)
    robot, D = _robot(case), 14 if case["arms"] == 2 else 7
    N = np.array([case["boxes"]])
    per = lambda N: 370 * D + 18 * robot.n_spheres + 300 + 20 * D * N
    if op == "steer":
        ev = case["edges"] * (case["steps"] + 1)
        return dict(bytes=4 * (case["edges"] * (3 * D + 2) + 10 * case["boxes"]), flops=float(ev * per(N)[0]))
    if case["seeds"] == 0:
        r = np.random.default_rng(4)
        P = case["problems"]
        S, T, N = r.integers(4, 65, P), r.choice([24, 32, 48], P), r.integers(5, 201, P)
    else:
        S, T = np.full(case["problems"], case["seeds"]), np.full(case["problems"], case["horizon"])
    rows, seeds = int((S * T).sum()), int(S.sum())
    K = case.get("K", 1)
    ev = {"steps": 1 + K * case.get("rounds", 0), "autograd": 2, "candidates": K,
          "particles": case.get("particles", 0) * case.get("rounds", 0),
          "solve": 2 + K * case.get("iters", 0)}.get(op, 1)
    out = {"candidates": K * (rows * D + 3 * seeds), "particles": 2 * rows * D + seeds * ev}.get(op, rows * D + 3 * seeds)
    return dict(bytes=4 * (rows * D * (2 if op == "candidates" else 1) + out + 10 * int(N.sum())),
                flops=float((S * T * per(N)).sum() * ev))


# ---------------------------------------------------------------------------
# the same results in 64 bits, from the definition of the cost

A = dict(a0=2000.0, a1=350.0, a2=100.0, a3=100.0, a6=5000.0, a7=50.0, a8=5000.0, a9=1.0, wb=5000.0, e2=0.1, wc=5000.0,
         eta=0.025, dt=0.25, ws=5000.0)
A.update({k: float(np.float32(A[k])) for k in ("e2", "eta")})


def _logcosh(x):
    x = x.abs()
    return x + torch.log1p(torch.exp(-2 * x)) - math.log(2.0)


def _norm(v):
    """Length with a zero gradient at zero."""
    n2 = (v * v).sum(-1)
    return torch.where(n2 > 0, torch.sqrt(torch.where(n2 > 0, n2, torch.ones_like(n2))), torch.zeros_like(n2))


class _World:
    def __init__(self, pose, dims, dev):
        t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=dev)
        w, x, y, z = (t(pose)[:, 3:] / t(pose)[:, 3:].norm(dim=1, keepdim=True)).T
        self.t, self.h = t(pose)[:, :3], t(dims) / 2
        self.R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                              1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                              1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)

    def sdf(self, p, i):
        """Signed distance of box-frame points to cuboid i and its gradient (box frame)."""
        a = p.abs() - self.h[i]
        q = a.clamp(min=0)
        out = q.norm(dim=-1)
        top = a.max(-1)
        s = torch.where(p >= 0, 1.0, -1.0).double()
        inner = torch.zeros_like(p).scatter_(-1, (a == top.values[..., None]).double().argmax(-1, keepdim=True), 1.0)
        far = out > 0
        g = torch.where(far[..., None], q / torch.where(far, out, torch.ones_like(out))[..., None], inner) * s
        return torch.where(far, out, top.values), g


def _dc(pen):
    eta = A["eta"]
    slope = ((pen + eta) / eta).clamp(0, 1)
    return torch.where(pen > 0, pen + eta / 2, slope * slope * eta / 2), slope


def _collision(world, c, r, before, after):
    """Summed collision cost of sphere centres c [n, m, 3] against the world,
    d cost / d centre, and the clearance; before / after: the centres at the
    neighbouring waypoints for the continuous check (or None), NaN where
    there is no neighbour."""
    cost, g, mc = torch.zeros(c.shape[0], dtype=c.dtype, device=c.device), torch.zeros_like(c), None
    mc = torch.full_like(cost, A["eta"])
    for i in range(len(world.h)):
        R = world.R[i]
        p = (c - world.t[i]) @ R
        s, gp = world.sdf(p, i)
        mc = torch.minimum(mc, (s - r).amin(1))
        v, sl = _dc(r - s)
        gb = -A["wc"] * sl[..., None] * gp
        for nb in (before, after):
            if nb is None:
                continue
            u = nb - c
            ln = u.norm(dim=-1)
            ok = ln > 0                                   # (NaN: no neighbour)
            u = torch.where(ok[..., None], u / ln[..., None], torch.zeros_like(u)) @ R
            rho = r + A["eta"]
            j = torch.where(s < rho, rho.expand_as(s), s - rho)
            for _ in range(4):
                on = ok & (j < 0.5 * ln)
                if not bool(on.any()):
                    break
                s2, g2 = world.sdf(p + j[..., None] * u, i)
                v2, sl2 = _dc(r - s2)
                v = v + torch.where(on, v2, torch.zeros_like(v2))
                gb = gb - A["wc"] * torch.where(on, sl2, torch.zeros_like(sl2))[..., None] * g2
                j = torch.where(on, j + torch.where(s2 - rho > 0, s2 - rho, rho.expand_as(s2)), j)
        cost = cost + A["wc"] * v.sum(1)
        g = g + gb @ R.T
    return cost, g, mc


class _Exact:
    def __init__(self, robot, swept, pairs=None):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.rb, self.swept = robot, swept
        t = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=self.dev)
        self.F = t(robot.fixed_tf).reshape(-1, 3, 4)
        self.sph, self.ee = t(robot.sphere), t(robot.ee_tf).reshape(-1, 3, 4)
        self.lo, self.hi = t(robot.q_lo), t(robot.q_hi)
        self.pairs = None if pairs is None else torch.as_tensor(np.asarray(pairs), dtype=torch.int64, device=self.dev)

    def fk(self, q):
        """Link rotations and origins, then sphere centres and tool frames, of q [n, D]."""
        R, p = [], []
        z, o = torch.zeros_like(q[:, 0]), torch.ones_like(q[:, 0])
        for l in range(self.rb.n_links):
            c, s = torch.cos(q[:, l]), torch.sin(q[:, l])
            Rz = torch.stack([c, -s, z, s, c, z, z, z, o], 1).reshape(-1, 3, 3)
            F = self.F[l]
            u = int(self.rb.parent[l])
            Rf, pf = (F[:, :3].expand(len(q), 3, 3), F[:, 3].expand(len(q), 3)) if u < 0 else \
                (R[u] @ F[:, :3], (R[u] @ F[:, 3]) + p[u])
            R.append(torch.matmul(Rf.contiguous(), Rz.contiguous()))
            p.append(pf)
        cs = [R[l] @ self.sph[m, :3] + p[l] for m, l in enumerate(self.rb.sphere_link)]
        ee = [(R[l] @ self.ee[e][:, :3], R[l] @ self.ee[e][:, 3] + p[l]) for e, l in enumerate(self.rb.ee_link)]
        return torch.stack(cs, 1) if cs else q.new_zeros((len(q), 0, 3)), ee

    @staticmethod
    def quat(R):
        """Unit quaternion (w x y z) by the largest of trace and diagonal."""
        tr = R[:, 0, 0] + R[:, 1, 1] + R[:, 2, 2]
        d = torch.stack([tr, R[:, 0, 0], R[:, 1, 1], R[:, 2, 2]], 1)
        k = d.argmax(1)
        out = R.new_zeros((len(R), 4))
        for b in range(4):
            i = torch.nonzero(k == b).flatten()
            if not len(i):
                continue
            M = R[i]
            e = lambda r, c: M[:, r, c]
            if b == 0:
                w = 0.5 * torch.sqrt(1 + tr[i])
                v = [w, (e(2, 1) - e(1, 2)) / (4 * w), (e(0, 2) - e(2, 0)) / (4 * w), (e(1, 0) - e(0, 1)) / (4 * w)]
            elif b == 1:
                x = 0.5 * torch.sqrt(1 + e(0, 0) - e(1, 1) - e(2, 2))
                v = [(e(2, 1) - e(1, 2)) / (4 * x), x, (e(0, 1) + e(1, 0)) / (4 * x), (e(0, 2) + e(2, 0)) / (4 * x)]
            elif b == 2:
                y = 0.5 * torch.sqrt(1 - e(0, 0) + e(1, 1) - e(2, 2))
                v = [(e(0, 2) - e(2, 0)) / (4 * y), (e(0, 1) + e(1, 0)) / (4 * y), y, (e(1, 2) + e(2, 1)) / (4 * y)]
            else:
                z = 0.5 * torch.sqrt(1 - e(0, 0) - e(1, 1) + e(2, 2))
                v = [(e(1, 0) - e(0, 1)) / (4 * z), (e(0, 2) + e(2, 0)) / (4 * z), (e(1, 2) + e(2, 1)) / (4 * z), z]
            out = out.index_copy(0, i, torch.stack(v, 1))
        return out

    def problem(self, world, q0, goal, T, x, grad=True, chunk=8192):
        """Cost [n], gradient [n, T, D] and clearance [n] of trajectories x [n, T, D] with
        starts q0 [n, D] and goals [n, n_ee, 7]."""
        parts, per = [], max(1, chunk // T)
        for a in range(0, len(x), per):
            parts.append(self._chunk(world, q0[a:a + per], goal[a:a + per], T, x[a:a + per], grad))
        return [torch.cat([p[i] for p in parts]) if parts[0][i] is not None else None for i in range(3)]

    def _chunk(self, world, q0, goal, T, x, grad):
        n, D = x.shape[0], x.shape[2]
        q = x.detach().requires_grad_(grad)
        with torch.set_grad_enabled(grad):
            c, ee = self.fk(q.reshape(-1, D))
            with torch.no_grad():
                before = after = None
                if self.swept and T > 1:
                    c0 = self.fk(q0)[0]
                    cc = c.reshape(n, T, -1, 3)
                    before = torch.cat([c0[:, None], cc[:, :-1]], 1).reshape(c.shape)
                    after = torch.cat([cc[:, 1:], torch.full_like(cc[:, :1], math.nan)], 1).reshape(c.shape)
                coll, gc, mc = _collision(world, c.detach(), self.sph[:, 3], before, after)
            cost = coll.reshape(n, T).sum(1)
            loss = (gc * c).sum()                          # (its derivative is the collision gradient)
            extra = torch.zeros_like(cost)
            if self.pairs is not None:
                i, j = self.pairs.T
                pen = self.sph[i, 3] + self.sph[j, 3] - _norm(c[:, i] - c[:, j])
                extra = extra + A["ws"] * pen.amax(1).clamp(min=0).reshape(n, T).sum(1)
            lo, hi, e2 = self.lo, self.hi, A["e2"]
            for v in (lo + e2 - q, q - (hi - e2)):         # distance into each limit band
                extra = extra + A["wb"] * torch.where(v > e2, v - e2 / 2, v.clamp(min=0) ** 2 / (2 * e2)).sum((1, 2))
            if T > 1:
                h = A["dt"]
                s = q0[:, None]
                X = torch.cat([s, s, s, q, q[:, -1:], q[:, -1:]], 1)
                m2, m1, z, p1, p2 = (X[:, k:k + T + 1] for k in range(5))
                v = (m2 - 8 * m1 + 8 * p1 - p2) / (12 * h)
                a = (-m2 + 16 * m1 - 30 * z + 16 * p1 - p2) / (12 * h * h)
                j = (-m2 + 2 * m1 - 2 * p1 + p2) / (2 * h ** 3)
                extra = extra + A["a6"] * _logcosh(A["a7"] * v[:, -1]).sum(1) + \
                    (A["a8"] * a * a + A["a9"] * j * j).sum((1, 2))
            last = torch.arange(n, device=q.device) * T + T - 1
            for e, (R, p) in enumerate(ee):
                g = goal[:, e]
                qt = self.quat(R[last])
                sg = torch.where((qt * g[:, 3:]).sum(1, keepdim=True) >= 0, 1.0, -1.0).double()
                extra = extra + A["a0"] * _logcosh(A["a2"] * _norm(g[:, :3] - p[last])) + \
                    A["a1"] * _logcosh(A["a3"] * _norm(g[:, 3:] - sg * qt))
            gr = torch.autograd.grad(loss + extra.sum(), q)[0] if grad else None
        return (cost + extra).detach(), gr, mc.reshape(n, T).amin(1)

    def batch(self, worlds, seeds, horizon, world, q0, goal, x, grad=True):
        """Per-seed cost, per-row gradient and per-seed clearance of a whole batch, the
        trajectories of one world and horizon together."""
        t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=self.dev)
        q0, goal = t(q0), t(goal).reshape(len(seeds), -1, 7)
        prob = np.repeat(np.arange(len(seeds)), seeds)
        T, w = horizon[prob], world[prob]
        row0 = np.cumsum(T) - T
        c, m = x.new_zeros(len(prob)), x.new_zeros(len(prob))
        g = torch.zeros_like(x) if grad else None
        for key in sorted(set(zip(w.tolist(), T.tolist()))):
            i = np.flatnonzero((w == key[0]) & (T == key[1]))
            rows = torch.as_tensor(row0[i][:, None] + np.arange(key[1]), device=self.dev)
            pi, si = torch.as_tensor(prob[i], device=self.dev), torch.as_tensor(i, device=self.dev)
            ci, gi, mi = self.problem(_World(*worlds.world(key[0]), self.dev), q0[pi], goal[pi], key[1], x[rows], grad)
            c[si], m[si] = ci, mi
            if grad:
                g[rows] = gi
        return c, g, m


def _philox(seed, k, it, q):
    """Philox-4x64 with ten rounds at counters {q, k, it, 0} and key {seed, 0}: [4, n] words."""
    M = [np.uint64(0xD2E7470EE14C6C93), np.uint64(0xCA5A826395121157)]
    W = [0x9E3779B97F4A7C15, 0xBB67AE8584CAA73B]
    lo32, s32 = np.uint64(0xFFFFFFFF), np.uint64(32)

    def mulhi(a, b):
        al, ah, bl, bh = a & lo32, a >> s32, b & lo32, b >> s32
        m1 = ah * bl + ((al * bl) >> s32)
        m2 = al * bh + (m1 & lo32)
        return ah * bh + (m1 >> s32) + (m2 >> s32)
    c = [q.astype(np.uint64), k.astype(np.uint64), np.full(q.shape, it, np.uint64), np.zeros(q.shape, np.uint64)]
    key = [int(seed), 0]
    for _ in range(10):
        h0, l0, h1, l1 = mulhi(c[0], M[0]), c[0] * M[0], mulhi(c[2], M[1]), c[2] * M[1]
        c = [h1 ^ c[1] ^ np.uint64(key[0]), l1, h0 ^ c[3] ^ np.uint64(key[1]), l0]
        key = [(a + b) % 2 ** 64 for a, b in zip(key, W)]
    return np.stack(c)


def _draws(seed, it, N, rows, D):
    n = rows * D
    nq = (n + 3) // 4
    k, q = np.meshgrid(np.arange(N), np.arange(nq), indexing="ij")
    w = _philox(seed, k.reshape(-1), it, q.reshape(-1))
    u1 = ((w >> np.uint64(41)).astype(np.float64) + 0.5) / 2 ** 23
    u2 = (((w >> np.uint64(9)) & np.uint64(0x7FFFFF)).astype(np.float64) + 0.5) / 2 ** 23
    z = np.sqrt(-2 * np.log(u1)) * np.cos(2 * np.pi * u2)
    return z.T.reshape(N, nq * 4)[:, :n].reshape(N, rows, D)


def _exact_steps(ex, args, x, alpha, rounds):
    """The L-BFGS direction and line search (Armijo and weak Wolfe) in 64 bits, every seed on its own."""
    worlds, seeds, horizon, world, q0, goal = args
    T = int(horizon[0])
    ev = lambda z: ex.batch(worlds, seeds, horizon, world, q0, goal, z)
    blk = lambda z: z.reshape(-1, T * z.shape[-1])
    c, g, mc = ev(x)
    n = len(c)
    hist = [[] for _ in range(n)]
    prev = None
    for it in range(rounds):
        X, G = blk(x), blk(g)
        d = torch.empty_like(X)
        for s in range(n):
            if prev is not None:
                sv, yv = X[s] - prev[0][s], G[s] - prev[1][s]
                if sv @ yv > 1e-10 * sv.norm() * yv.norm() and sv @ yv > 0:
                    hist[s] = (hist[s] + [(sv, yv)])[-4:]
            q, al = G[s].clone(), []
            for sv, yv in reversed(hist[s]):
                al.append((sv @ q) / (sv @ yv))
                q = q - al[-1] * yv
            if hist[s]:
                sv, yv = hist[s][-1]
                q = q * ((sv @ yv) / (yv @ yv))
            else:
                gi = float(G[s].abs().max())
                q = q * (min(1.0, 0.1 / gi) if gi > 0 else 1.0)
            for (sv, yv), a in zip(hist[s], reversed(al)):
                q = q + (a - (yv @ q) / (sv @ yv)) * sv
            d[s] = -q
        prev = (X.clone(), G.clone())
        g0d = (G * d).sum(1)
        xs, cs, gs, ms = [], [], [], []
        for a in alpha:
            z = torch.minimum(torch.maximum(x + a * d.reshape(x.shape), ex.lo), ex.hi)
            ck, gk, mk = ev(z)
            xs.append(z), cs.append(ck), gs.append(gk), ms.append(mk)
        best = torch.zeros(n, dtype=torch.int64, device=c.device)
        for k in range(1, len(alpha)):
            gd = (blk(gs[k]) * d).sum(1)
            ok = (cs[k] <= c + 1e-4 * alpha[k] * g0d) & (gd >= 0.9 * g0d)
            best = torch.where(ok, torch.full_like(best, k), best)
        s = torch.arange(n, device=c.device)
        x = torch.stack([blk(z) for z in xs])[best, s].reshape(x.shape)
        g = torch.stack([blk(z) for z in gs])[best, s].reshape(x.shape)
        c, mc = torch.stack(cs)[best, s], torch.stack(ms)[best, s]
    return x, c, g, None, mc


def exact(case, seed):
    op = case["op"]
    if op == "solve":
        return None                                        # (an iteration's rounding grows over the solve)
    if op == "knn":
        nodes, queries = (torch.as_tensor(a, dtype=torch.float64) for a in _knn_inputs(case, seed))
        if torch.cuda.is_available():
            nodes, queries = nodes.cuda(), queries.cuda()
        k = min(case["k"], len(nodes))
        d2 = torch.cat([((queries[a:a + 256, None] - nodes[None]) ** 2).sum(2).topk(k, largest=False).values
                        for a in range(0, len(queries), 256)])
        pad = d2.new_full((len(d2), case["k"] - k), math.inf)
        return None, torch.cat([d2, pad], 1)
    if op == "steer":
        robot, worlds, _, _, _ = _scene(case, seed)
        ex = _Exact(robot, 0)
        a, b, res = _steer_inputs(case, seed, robot)
        n = np.floor(np.abs(b - a).max(1) / np.float32(res)).astype(int) + 1
        t = lambda v: torch.as_tensor(v, dtype=torch.float64, device=ex.dev)
        a, b, nt = t(a), t(b), t(n)
        i = torch.arange(case["steps"] + 1, dtype=torch.float64, device=ex.dev)
        f = torch.where(nt[:, None] <= case["steps"], torch.minimum(i[None], nt[:, None]) / nt[:, None], 0.0)
        pts = a[:, None] + f[..., None] * (b - a)[:, None]
        world = _World(*worlds.world(0), ex.dev)
        flat = pts.reshape(-1, a.shape[1])
        mc = torch.cat([_collision(world, ex.fk(flat[k:k + 8192])[0], ex.sph[:, 3], None, None)[2]
                        for k in range(0, len(flat), 8192)]).reshape(pts.shape[:2])
        bad = (mc < 0) | (pts < ex.lo).any(2) | (pts > ex.hi).any(2)
        bad = torch.cat([bad, torch.ones_like(bad[:, :1])], 1)
        first = torch.minimum(bad.double().argmax(1), nt.long() + 1)
        last = torch.where(nt <= case["steps"], first - 1, torch.full_like(first, -2))
        reach = torch.where((last >= 0)[:, None], pts[torch.arange(len(a), device=ex.dev), last.clamp(min=0)], a)
        return reach, None, (reach - a).norm(dim=1)
    robot, worlds, seeds, horizon, world, q0, goal, x, d = _inputs(case, seed)
    ex = _Exact(robot, case["swept"], wl.self_pairs(robot) if case.get("self_pairs") else None)
    args = (worlds, seeds, horizon, world, q0, goal)
    alpha = [float(np.float32(v)) for v in ALPHAS.get(case.get("K", 1), (1.0,))]
    X = torch.as_tensor(x, dtype=torch.float64, device=ex.dev)
    S = np.repeat(np.arange(len(seeds)), seeds)
    if op == "cost_grad":
        return ex.batch(*args, X)
    if op == "autograd":
        c, g, _ = ex.batch(*args, X)
        w = np.random.default_rng(seed).uniform(0.5, 1.5, len(S)).astype(np.float32)
        return c, g * torch.as_tensor(np.repeat(w, horizon[S]), dtype=torch.float64, device=ex.dev)[:, None]
    if op == "steps":
        return _exact_steps(ex, args, X, alpha, case["rounds"])
    if op == "candidates":
        Dv = torch.as_tensor(d, dtype=torch.float64, device=ex.dev)
        cost, gd, grad, mc = [], [], [], []
        at = torch.as_tensor(np.repeat(np.arange(len(S)), horizon[S]), device=ex.dev)
        for a in alpha:
            c, g, m = ex.batch(*args, torch.minimum(torch.maximum(X + a * Dv, ex.lo), ex.hi))
            cost.append(c), grad.append(g), mc.append(m)
            gd.append(torch.zeros_like(c).index_add_(0, at, (g * Dv).sum(1)))
        return torch.stack(cost), torch.stack(gd), torch.stack(grad), torch.stack(mc)
    # particles
    N, T, Sn = case["particles"], int(horizon[0]), int(seeds[0])
    W = _World(*worlds.world(0), ex.dev)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=ex.dev)
    var = torch.full_like(X, float(np.float32(0.05 ** 2)))
    costs = []
    for it in range(case["rounds"]):
        e = t(_draws(seed, it, N, len(X), X.shape[1]))
        th = torch.minimum(torch.maximum(X + torch.sqrt(var) * e, ex.lo), ex.hi)        # [N, rows, D]
        c = ex.problem(W, t(q0[:1]).expand(N * Sn, -1), t(goal[:1]).reshape(1, -1, 7).expand(N * Sn, -1, -1), T,
                       th.reshape(N * Sn, T, -1), grad=False)[0]
        c = c.reshape(N, Sn)
        costs.append(c.T)
        w = torch.exp(-(c - c.amin(0)) / (0.1 * (c.amax(0) - c.amin(0)) + 1e-12))
        w = (w / w.sum(0)).repeat_interleave(T, 1)[..., None]                            # [N, rows, 1]
        k_mu, k_s = float(np.float32(0.9)), 0.5
        X, var = (1 - k_mu) * X + k_mu * (w * th).sum(0), (1 - k_s) * var + k_s * (w * (th - X) ** 2).sum(0)
    return X, var, torch.stack(costs)
