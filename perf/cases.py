"""Performance cases: what programs that use this framework have it do, through its public entry points.

A case is a dict of plain values. ``kind`` names the call a program makes:

  solve     one solve from a new initial state (``Solver.solve_x0``), or of new q, l, u
            (``Solver.update_device`` and ``Solver.solve``) for a dense QP
  sequence  ``count`` solves from ``count`` initial states in one launch (``Solver.solve_sequence``)
  loop      a closed control loop of ``steps`` MPC steps of ``budget`` iterations (``Solver.closed_loop``)
  batch     ``batch`` instances of one family solved together (``Solver.solve_x0`` of a batched handle)
  serve     a serving handle's slots: requests loaded and admitted cold, a step, more requests
            admitted warm from a slot's solution shifted by one stage, another step
  setup     a new problem family: ``Solver(...)`` (factorisations of every penalty) and its first solve

Problems are random linear MPC (condensed, LQR-preconditioned: ``nx`` states, ``nu`` controls,
``N`` stages, control limits and optionally state limits) or random dense QPs with a quarter of n
equality and a quarter inequality rows. A family's matrices are fixed by ``family``; initial
states (``scale`` times uniform) or vectors come from the seed. At scale 1 an MPC solve stops at
its first check; larger scales make the limits bind and the penalty move.
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2311_18056_amd as rq

DEV = "cuda"
F64 = torch.float64


# ------------------------------------------------------------------------------------------
# Problems (FP64, on the host; built once per family)


def _riccati(A, B, Q, R):
    """LQR gain of the infinite-horizon problem by the doubling form of the Riccati recursion."""
    n = A.shape[0]
    eye = np.eye(n)
    a, g, h = A.copy(), B @ np.linalg.solve(R, B.T), Q.copy()
    for _ in range(60):
        w = np.linalg.inv(eye + g @ h)
        h1 = h + a.T @ h @ w @ a
        g = g + a @ w @ g @ a.T
        a = a @ w @ a
        done = np.max(np.abs(h1 - h)) <= 1e-14 * np.max(np.abs(h1))
        h = 0.5 * (h1 + h1.T)
        g = 0.5 * (g + g.T)
        if done:
            break
    return np.linalg.solve(R + B.T @ h @ B, B.T @ h @ A)


@functools.lru_cache(maxsize=4)
def _mpc(nx, nu, N, x_box, family):
    """P, A, F, E, lo, hi, Ad, Bd of a condensed MPC family; x_box 0: control limits only."""
    rng = np.random.default_rng(family)
    A0 = rng.standard_normal((nx, nx))
    Ad = A0 * ((1.02 if x_box else 1.05) / np.max(np.abs(np.linalg.eigvals(A0))))
    Bd = rng.standard_normal((nx, nu))
    if x_box:  # the humanoid-shaped family: sparse B, uneven state weights, cheap controls
        Bd *= rng.random((nx, nu)) < 0.3
        Q, R = np.diag(rng.uniform(1.0, 10.0, nx)), 0.01 * np.eye(nu)
    else:
        Q, R = np.eye(nx), 0.1 * np.eye(nu)
    K = _riccati(Ad, Bd, Q, R)
    Ab = Ad - Bd @ K
    n = N * nu
    Sx, Mx = np.zeros((N + 1, nx, n)), np.zeros((N + 1, nx, nx))
    Mx[0] = np.eye(nx)
    for k in range(N):
        Sx[k + 1] = Ab @ Sx[k]
        Sx[k + 1][:, k * nu:(k + 1) * nu] += Bd
        Mx[k + 1] = Ab @ Mx[k]
    Su, Mu = np.matmul(-K, Sx[:N]), np.matmul(-K, Mx[:N])
    for k in range(N):
        Su[k][:, k * nu:(k + 1) * nu] += np.eye(nu)
    Su, Mu, Sx, Mx = Su.reshape(n, n), Mu.reshape(n, nx), Sx[1:].reshape(N * nx, n), Mx[1:].reshape(N * nx, nx)
    QSx = np.tile(np.diag(Q), N)[:, None] * Sx
    P = Su.T @ (R[0, 0] * Su) + Sx.T @ QSx
    F = Su.T @ (R[0, 0] * Mu) + QSx.T @ Mx
    A, E, lim = Su, Mu, np.ones(n)
    if x_box:
        A, E, lim = np.vstack([Su, Sx]), np.vstack([Mu, Mx]), np.concatenate([lim, x_box * np.ones(N * nx)])
    return 0.5 * (P + P.T), A, F, E, -lim, lim, Ad, Bd


@functools.lru_cache(maxsize=4)
def _dense(n, family):
    rng = np.random.default_rng(family)
    m = 2 * max(1, n // 4)
    M = rng.standard_normal((n, n))
    P = M.T @ M / n + 1e-2 * np.eye(n)
    return 0.5 * (P + P.T), rng.standard_normal((m, n)) / math.sqrt(n)


def _dense_vectors(A, seed):
    """q, l, u of a feasible dense QP: the first half of the rows are equalities."""
    rng = np.random.default_rng(seed)
    m, n = A.shape
    q, Ax, w = rng.standard_normal(n), A @ rng.standard_normal(n), rng.uniform(0.0, 1.0, m)
    w[:m // 2] = 0.0
    return q, Ax - w, Ax + w


def _problem(case, seed):
    if case["kind"] == "setup":  # a new model each time: its matrices come from the seed
        return _mpc(case["nx"], case["nu"], case["N"], case["x_box"], seed)
    return _mpc(case["nx"], case["nu"], case["N"], case["x_box"], case["family"])


def _x0(case, count, seed):
    rng = np.random.default_rng(seed)
    return case["scale"] * rng.uniform(-1.0, 1.0, (count, case["nx"]))


def _settings(case):
    if "dense" in case:
        s = dict(n_rho=8, eps_abs=1e-6, eps_rel=1e-6, max_iter=20000)
    elif case["kind"] == "loop":
        s = dict(n_rho=8, eps_abs=0.0, eps_rel=0.0, max_iter=case["budget"])
    else:
        # an iteration budget, as a controller with a deadline sets it
        s = dict(n_rho=case["n_rho"], eps_abs=1e-3, eps_rel=1e-3, max_iter=100 if case["kind"] == "batch" else 150)
    return dict(s, precision=case["precision"], check_interval=25)


# ------------------------------------------------------------------------------------------
# The cases


def listed():
    mpc = dict(x_box=0.0, n_rho=8, scale=1.0)
    return [
        # the smallest controller (n = m = 20, one penalty, FP64), one solve per control tick
        dict(name="mpc20_fp64_solve", kind="solve", nx=6, nu=2, N=10, family=0, precision="fp64", **dict(mpc, n_rho=1)),
        # a small dense QP to 1e-6, as a program with changing vectors solves it
        dict(name="dense60_fp64_solve", kind="solve", dense=60, family=600000, precision="fp64"),
        # the first size past 128 rows (n = 104, m = 52)
        dict(name="dense104_fp64_solve", kind="solve", dense=104, family=1040000, precision="fp64"),
        # the largest dense QP of the paper's range
        dict(name="dense2000_fp64_solve", kind="solve", dense=2000, family=20000000, precision="fp64"),
        # the n = m = 1600 controller, one solve per tick: latency
        dict(name="mpc1600_fp32_solve", kind="solve", nx=120, nu=40, N=40, family=1, precision="fp32", **mpc),
        # the same family, initial states queued and solved in one launch, limits binding
        dict(name="mpc1600_fp32_sequence", kind="sequence", nx=120, nu=40, N=40, family=1, precision="fp32", count=20,
             **dict(mpc, scale=20.0)),
        # the humanoid-shaped controller: control and state limits (n = 600, m = 1800)
        dict(name="mpc600x1800_fp32_sequence", kind="sequence", nx=60, nu=30, N=20, family=2, precision="fp32",
             count=20, **dict(mpc, x_box=2.0)),
        # simulation in the loop, two iterations per step (n = m = 400)
        dict(name="loop400_fp64", kind="loop", nx=30, nu=10, N=40, x_box=0.0, scale=5.0, family=70, precision="fp64",
             steps=100, budget=2),
        # many initial states of one large family at once (sampling, Monte Carlo): throughput
        dict(name="batch4096_mpc1600_bf16x3", kind="batch", nx=120, nu=40, N=40, family=1, precision="bf16x3",
             batch=4096, **mpc),
        # a ragged batch of a middle-sized family with FP32 products
        dict(name="batch333_mpc800_fp32", kind="batch", nx=60, nu=20, N=40, family=41, precision="fp32", batch=333,
             **dict(mpc, scale=5.0)),
        # a serving tick of the smallest served family: cold and warm requests in 128 slots
        dict(name="serve128_mpc200_bf16x3", kind="serve", nx=15, nu=5, N=40, family=40, precision="bf16x3", batch=128,
             cold=75, warm=32, **dict(mpc, scale=10.0)),
        # a model linearised anew: every penalty's factorisation, then the first solve
        dict(name="setup600x1800_fp32", kind="setup", nx=60, nu=30, N=20, precision="fp32", **dict(mpc, x_box=2.0)),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.randrange(1 << 20)
    pick = rng.random()
    if pick < 0.25:
        return dict(kind="solve", dense=_log(rng, 10, 2000), family=family, precision="fp64")
    if pick < 0.5:
        case = dict(kind="solve", precision=rng.choice(["fp32", "fp32", "fp64"]))
    elif pick < 0.62:
        case = dict(kind="sequence", precision="fp32", count=rng.randrange(2, 25))
    elif pick < 0.72:
        case = dict(kind="loop", precision="fp64", steps=rng.randrange(20, 120), budget=rng.choice([1, 2, 15]))
    elif pick < 0.84:
        case = dict(kind="batch", precision=rng.choice(["bf16x3", "fp32"]), batch=_log(rng, 2, 2048))
    elif pick < 0.94:
        slots = rng.choice([48, 64, 128, 256])
        cold = rng.randrange(1, slots // 2)
        case = dict(kind="serve", precision="bf16x3", batch=slots, cold=cold, warm=rng.randrange(1, slots - cold))
    else:
        case = dict(kind="setup", precision="fp32")
    N = rng.randrange(10, 41)
    top = 700 if case["kind"] in ("loop", "setup") or case["precision"] == "fp64" else 1600
    n = _log(rng, 20 if top == 700 else 60, 800 if case["kind"] == "serve" else top)
    nu = max(1, round(n / N))
    x_box = 2.0 if rng.random() < 0.25 and n <= 600 and case["kind"] != "loop" else 0.0
    case.update(nx=2 * nu if x_box else 3 * nu, nu=nu, N=N, x_box=x_box)
    if case["kind"] != "loop":
        case["n_rho"] = rng.choice([1, 8, 8])
    # a single fixed penalty and large samples go with states near the nominal one
    near = x_box or case.get("n_rho") == 1 or case.get("batch", 1) > 256
    near = near or (case["kind"] == "batch" and n > 800)
    case["scale"] = 1.0 if near else rng.choice([1.0, 5.0]) if case["kind"] == "loop" else rng.choice([1.0, 5.0, 10.0])
    if case["kind"] != "setup":
        case["family"] = family
    return case


# ------------------------------------------------------------------------------------------


def _size(case):
    if "dense" in case:
        return case["dense"], 2 * max(1, case["dense"] // 4)
    n = case["nu"] * case["N"]
    return n, n + (case["nx"] * case["N"] if case["x_box"] else 0)


def _f64(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=F64, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if "dense" in case:
        P, A = _dense(case["dense"], case["family"])
        q, l, u = _dense_vectors(A, seed)
        s = rq.Solver(P, q, A, l, u, **_settings(case))
        return dict(kind="vectors", solver=s, q=_f64(q), l=_f64(l), u=_f64(u))
    P, A, F, E, lo, hi, Ad, Bd = _problem(case, seed)
    count = {"sequence": case.get("count"), "batch": case.get("batch")}.get(kind, 1)
    if kind == "serve":
        count = case["cold"] + case["warm"]
    x0 = _x0(case, count, seed)
    if kind == "setup":
        q, l, u = F @ x0[0], lo - E @ x0[0], hi - E @ x0[0]
        return dict(kind=kind, data=(P, q, A, l, u), settings=_settings(case))
    B = case["batch"] if kind in ("batch", "serve") else 1
    q0, l0, u0 = np.zeros((B, P.shape[0])), np.tile(lo, (B, 1)), np.tile(hi, (B, 1))
    more = dict(engine="batch" if kind in ("batch", "serve") else "single")
    if B == 1:
        q0, l0, u0 = q0[0], l0[0], u0[0]
    s = rq.Solver(P, q0, A, l0, u0, **more, **_settings(case))
    s.set_parametric(F, E, lo, hi)
    st = dict(kind=kind, solver=s, x0=_f64(x0))
    if kind == "sequence":
        st["out"] = s.sequence_slots(count)
    elif kind == "loop":
        st.update(x0=st["x0"][0].clone(), Ad=_f64(Ad), Bd=_f64(Bd), nu=case["nu"], steps=case["steps"])
        st["out"] = s.sequence_slots(case["steps"])
        st["out"]["traj_x"] = torch.zeros(case["steps"] + 1, case["nx"], dtype=F64, device=DEV)
        st["out"]["traj_u"] = torch.zeros(case["steps"], case["nu"], dtype=F64, device=DEV)
    elif kind == "serve":
        c = case["cold"]
        st.update(cold=list(range(c)), warm=list(range(c, c + case["warm"])), stage=case["nu"],
                  x0c=st["x0"][:c].clone(), x0w=st["x0"][c:].clone())
    return st


def _results(s):
    return dict(x=s.x, z=s.z, y=s.y, iterations=s.iterations, status=s.status, rho_index=s.rho_index)


def run(state):
    kind = state["kind"]
    if kind == "setup":
        s = rq.Solver(*state["data"], **state["settings"])
        s.solve()
        out = _results(s)
        s.close()
        return out
    s = state["solver"]
    if kind == "vectors":
        s.update_device(state["q"], state["l"], state["u"])
        s.solve()
    elif kind == "sequence":
        o = s.solve_sequence(state["x0"], out=state["out"])
        return {k: o[k] for k in ("x", "z", "y", "iterations", "status", "rho_index")}
    elif kind == "loop":
        o = s.closed_loop(state["x0"], state["steps"], state["Ad"], state["Bd"], state["nu"], out=state["out"])
        return {k: o[k] for k in ("x", "z", "y", "iterations", "status", "rho_index", "traj_x", "traj_u")}
    elif kind == "serve":
        s.load_slots_x0(state["cold"], state["x0c"])
        s.admit(state["cold"])
        s.step(1)
        s.load_slots_x0(state["warm"], state["x0w"])
        s.admit(state["warm"], src_slot=0, shift_x=state["stage"], shift_y=state["stage"])
        s.step(2)
    else:
        s.solve_x0(state["x0"])
    return _results(s)


def work(case):
    """One pass' necessary bytes and operations. An iteration or a check multiplies the n x n and
    twice the n x m entries (the two-product form); a solve has at least one check interval, a
    binding or 1e-6 one about two. Matrices are read once per pass, vectors per instance."""
    n, m = _size(case)
    kind, nx = case["kind"], case.get("nx", 0)
    es = 8 if case["precision"] == "fp64" else 4
    entries = n * n + 2 * n * m
    count = case.get("count") or case.get("batch") or 1
    layers = 78 if "dense" in case else 26 if case.get("scale", 1.0) <= 1.0 else 52
    if kind == "loop":
        count, layers = case["steps"], case["budget"]
    elif kind == "serve":
        count = case["cold"] + case["warm"]
    flops = 2.0 * entries * layers * count
    per = (n + 2 * m) * es + (8 * (n + 2 * m) if "dense" in case else 8 * nx)
    byts = float(entries * es * (1 if kind == "loop" else 2) + 8 * (n + m) * nx + count * per)
    if kind == "setup":
        nr = case["n_rho"]
        flops += 2.0 * n * n * m + nr * (2.0 * n ** 3 + 2.0 * n * n * m + 2.0 * n * m * m)
        byts = 8.0 * (n * n + m * n) + nr * es * float(n + m) ** 2 + per
    return {"bytes": byts, "flops": flops}


# ------------------------------------------------------------------------------------------
# The same solves in 64 bits with plain torch (textbook ADMM with over-relaxation: two products per
# iteration with the explicit inverse, the clamp, the dual update; residual test and nearest grid
# penalty every 25 iterations).


class _Admm:
    def __init__(self, P, A, eq, n_rho, eps):
        self.P, self.A, self.eps, self.ci = _f64(P), _f64(A), eps, 25
        self.om = torch.where(_f64(eq) > 0, 1e3, 1.0)
        grid = np.logspace(-3, 3, n_rho) if n_rho > 1 else np.array([0.1])
        self.grid = torch.tensor(grid, dtype=F64, device=DEV)
        self.j0 = int(np.argmin(np.abs(np.log(grid) - np.log(0.1))))
        self.cache = {}

    def inverse(self, j):
        if j not in self.cache:
            K = self.P + 1e-6 * torch.eye(self.P.shape[0], dtype=F64, device=DEV)
            K = K + self.A.t().contiguous() @ ((self.grid[j] * self.om)[:, None] * self.A)
            self.cache[j] = torch.linalg.inv(0.5 * (K + K.t()))
        return self.cache[j]

    def solve(self, q, l, u, most, warm=None):
        """Rows of q, l, u are instances; at most `most` iterations (a check only at multiples of
        25). Returns x, z, y and penalty indices."""
        P, A = self.P, self.A
        At = A.t().contiguous()
        B, m = l.shape
        if warm is None:
            x, y = torch.zeros_like(q), torch.zeros_like(l)
            z, j = torch.zeros_like(l), torch.full((B,), self.j0, device=DEV)
        else:
            x, y, j = warm[0].clone(), warm[1].clone(), warm[2].clone()
            z = x @ At
        live = torch.ones(B, dtype=torch.bool, device=DEV)
        k = 0
        while k < most and bool(live.any()):
            stop = min(most, (k // self.ci + 1) * self.ci)
            for g in torch.unique(j[live]).tolist():
                at = torch.nonzero(live & (j == g)).reshape(-1)
                D, rho = self.inverse(g), (self.grid[g] * self.om)[None, :]
                xs, zs, ys, qs, ls, us = x[at], z[at], y[at], q[at], l[at], u[at]
                for _ in range(stop - k):
                    xt = (1e-6 * xs - qs + (rho * zs - ys) @ A) @ D
                    t = 1.6 * (xt @ At) - 0.6 * zs + ys / rho
                    xs = 1.6 * xt - 0.6 * xs
                    zs = torch.minimum(torch.maximum(t, ls), us)
                    ys = rho * (t - zs)
                x[at], z[at], y[at] = xs, zs, ys
            k = stop
            if k % self.ci:
                break
            Ax, Px, Ay = x @ At, x @ P, y @ A
            top = lambda v: v.abs().amax(1)  # noqa: E731
            rp, rd = top(Ax - z), top(Px + q + Ay)
            np_, nd = torch.maximum(top(Ax), top(z)), torch.maximum(torch.maximum(top(Px), top(Ay)), top(q))
            if self.eps > 0:
                live &= ~((rp <= self.eps * (1 + np_)) & (rd <= self.eps * (1 + nd)))
            want = self.grid[j] * torch.sqrt(rp * nd.clamp_min(1e-4) / (rd * np_.clamp_min(1e-4)))
            near = (self.grid.log()[None, :] - want.log()[:, None]).abs().argmin(1)
            j = torch.where(live & (rp > 0) & (rd > 0), near, j)
        return x, z, y, j


def _named(r):
    return dict(x=r[0], z=r[1], y=r[2], iterations=None, status=None, rho_index=None)


def exact(case, seed):
    kind, st = case["kind"], _settings(case)
    if "dense" in case:
        P, A = _dense(case["dense"], case["family"])
        q, l, u = _dense_vectors(A, seed)
        a = _Admm(P, A, l == u, st["n_rho"], st["eps_abs"])
        return _named(a.solve(_f64(q)[None], _f64(l)[None], _f64(u)[None], st["max_iter"]))
    P, A, F, E, lo, hi, Ad, Bd = _problem(case, seed)
    a = _Admm(P, A, lo == hi, st["n_rho"], st["eps_abs"])
    Ft, Et, lo, hi = _f64(F.T), _f64(E.T), _f64(lo), _f64(hi)
    vec = lambda x0: (x0 @ Ft, lo - x0 @ Et, hi - x0 @ Et)  # noqa: E731
    if kind == "loop":
        x0, nu, warm, got = _f64(_x0(case, 1, seed)), case["nu"], None, []
        Adt, Bdt = _f64(Ad.T), _f64(Bd.T)
        tx, tu = [x0], []
        for _ in range(case["steps"]):
            r = a.solve(*vec(x0), case["budget"], warm)
            warm = (r[0], r[2], r[3])
            tu.append(r[1][:, :nu] + (x0 @ Et)[:, :nu])
            x0 = x0 @ Adt + tu[-1] @ Bdt
            tx.append(x0)
            got.append(r)
        out = _named([torch.cat([g[i] for g in got]) for i in range(3)])
        return dict(out, traj_x=torch.cat(tx), traj_u=torch.cat(tu))
    if kind == "serve":
        c, w, s = case["cold"], case["warm"], case["nu"]
        x0 = _f64(_x0(case, c + w, seed))
        first = a.solve(*vec(x0[:1]), 25)
        shift = lambda v: torch.cat([v[:, s:], torch.zeros_like(v[:, :s])], 1).repeat(w, 1)  # noqa: E731
        rc = a.solve(*vec(x0[:c]), 75)
        rw = a.solve(*vec(x0[c:]), 50, (shift(first[0]), shift(first[2]), first[3].repeat(w)))
        rest = case["batch"] - c - w
        return _named([torch.cat([p, r, torch.zeros(rest, p.shape[1], dtype=F64, device=DEV)])
                       for p, r in zip(rc[:3], rw[:3])])
    count = {"sequence": case.get("count"), "batch": case.get("batch")}.get(kind, 1)
    return _named(a.solve(*vec(_f64(_x0(case, count, seed))), st["max_iter"]))
