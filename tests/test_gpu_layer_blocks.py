"""The persistent layer kernel on few workgroups: blocks of more rows than the usual instantiation keeps
in registers, up to the 64 a workgroup may own. A row's products are summed in the same order wherever
the row is kept and whichever workgroup owns it, so with a fixed penalty and a fixed number of
iterations every grid returns the default grid's bits: plain, Ruiz-scaled and closed-loop solves."""

import numpy as np
import pytest

import oracle
from oracle import admm
from workloads import random_mpc, random_qp, x0_batch

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-9, "fp32": 1e-4}  # the per-iterate tolerances of the FP64 and FP32 kernels

# rows per workgroup around the 13, 16 and 32 that the instantiations keep in registers, passes of 8 more
# each, and the most that are accepted
ROWS = (13, 14, 16, 17, 21, 22, 24, 25, 29, 30, 32, 33, 40, 41, 64)


@pytest.mark.parametrize("prec,n,m", [
    ("fp32", 20, 20), ("fp32", 70, 330), ("fp32", 300, 469), ("fp32", 201, 2000), ("fp32", 201, 3200),
    ("fp64", 20, 20), ("fp64", 70, 186), ("fp64", 300, 500), ("fp64", 201, 2000),
])
def test_every_grid_returns_the_same_iterates(prec, n, m):
    import paper_2311_18056_amd as rq

    L = n + m
    P, q, A, l, u = random_qp(n, 0, m, seed=3 * n + m)
    kw = dict(n_rho=1, eps_abs=0.0, eps_rel=0.0, max_iter=57)
    sol = rq.Solver(P, q, A, l, u, precision=prec, engine="single", **kw)
    first = None
    for grid in sorted({min(-(-L // r), 256) for r in ROWS}, reverse=True):
        print(f"\n{prec}: n + m = {L}, {grid} workgroups of up to {-(-L // grid)} rows", flush=True)
        sol.set_launch(grid)
        sol.solve()
        res = sol.result()
        assert res["iterations"] == 57 and res["status"] == rq.RQP_MAX_ITER
        if first is None:
            first = res
            ref = oracle.solve(P, q, A, l, u, admm.Settings(**kw))
            for name in ("x", "z", "y"):
                b = getattr(ref, name)
                assert np.max(np.abs(res[name] - b)) <= TOL[prec] * max(np.max(np.abs(b)), 1.0), name
        for name in ("x", "z", "y"):
            assert np.array_equal(res[name], first[name]), (grid, name)
    sol.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("scaling", [0, 10])  # closed loops; scaled sequences (the same instantiations)
def test_every_grid_returns_the_same_loops_and_scaled_solves(prec, scaling):
    import torch

    import paper_2311_18056_amd as rq

    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")  # noqa: E731
    for nx, nu, N in ((15, 5, 40), (30, 10, 40)):  # 400 and 800 rows
        prob = random_mpc(nx, nu, N, seed=90 + nu)
        xs = 5.0 * x0_batch(nx, 3, 45)
        q, l, u = prob.instance(xs[0])
        kw = dict(n_rho=1, eps_abs=0.0, eps_rel=0.0, max_iter=31, scaling=scaling)
        sol = rq.Solver(prob.P, q, prob.A, l, u, precision=prec, engine="single", **kw)
        sol.set_parametric(prob.F, prob.E, prob.lo, prob.hi)
        L, first = q.size + l.size, None
        for rows in (8, 13, 14, 17, 30, 33, 64):
            grid = -(-L // rows)
            print(f"\n{prec}, scaling {scaling}: n + m = {L}, {grid} workgroups", flush=True)
            sol.set_launch(grid)
            if scaling:
                out = sol.solve_sequence(dev(xs))
            else:
                out = sol.closed_loop(dev(xs[0]), 5, dev(prob.A_dyn), dev(prob.B), nu)
            out = {k: v.cpu().numpy() for k, v in out.items() if k in ("x", "z", "y", "status", "traj_x", "traj_u")}
            assert np.all(out["status"] == rq.RQP_MAX_ITER)
            first = first or out
            for name in out:
                assert np.array_equal(out[name], first[name]), (grid, name)
        sol.close()
