"""The persistent layer kernel at the edges of its layouts: numbers of rows where the lanes and the
columns per lane change, row blocks that reach from registers into LDS and memory, and checks whose
rows are partly kept in LDS. Per iterate against the FP64 oracle with the penalty schedule replayed,
two checks and a ragged end."""

import numpy as np
import pytest

import oracle
from oracle import admm
from workloads import random_qp

TOL = {"fp64": 1e-9, "fp32": 1e-4}  # the per-iterate tolerances of the FP64 and FP32 kernels


@pytest.fixture(scope="module")
def rq():
    import paper_2311_18056_amd as rq

    return rq


@pytest.mark.gpu
@pytest.mark.parametrize("prec,n,m_eq,m_in,grid", [
    # one wave of columns; one row past 512, 1024; five columns per lane and one row past it
    ("fp32", 70, 0, 59, 0), ("fp32", 300, 0, 213, 0), ("fp32", 700, 0, 325, 0), ("fp32", 1300, 0, 1261, 0),
    # one row past five columns of 1024 lanes, 21 rows per workgroup: registers and LDS
    ("fp32", 2700, 0, 2421, 0),
    # 63 rows per workgroup: registers, LDS and memory
    ("fp32", 1300, 0, 1261, 41), ("fp64", 300, 20, 193, 9),
    # two columns per lane; one row past two columns, and past three, of 1024 lanes
    ("fp64", 70, 10, 49, 0), ("fp64", 500, 20, 505, 0), ("fp64", 1050, 20, 979, 0), ("fp64", 1600, 30, 1443, 0),
    # many more constraint rows than variables
    ("fp32", 41, 0, 600, 0),
])
def test_layer_shapes(rq, prec, n, m_eq, m_in, grid):
    P, q, A, l, u = random_qp(n, m_eq, m_in, seed=7 * n + m_in)
    sol = rq.Solver(P, q, A, l, u, precision=prec, n_rho=8, eps_abs=0.0, eps_rel=0.0, max_iter=57)
    if grid:
        sol.set_launch(grid)
    sol.solve()
    res = sol.result()
    sol.close()
    s = admm.Settings(n_rho=8, eps_abs=0.0, eps_rel=0.0, max_iter=57)
    ref = oracle.solve(P, q, A, l, u, s, rho_replay=res["rho_hist"])
    assert res["iterations"] == 57 and res["status"] == rq.RQP_MAX_ITER
    for name in ("x", "z", "y"):
        a, b = res[name], getattr(ref, name)
        assert np.max(np.abs(a - b)) <= TOL[prec] * max(np.max(np.abs(b)), 1.0), name
    for name in ("prim_res", "dual_res"):
        b = np.asarray(getattr(ref, name))
        # residuals are differences of terms of order one: absolute at the iterates' tolerance times
        # the largest row sum of the check matrix
        scale = max(np.abs(np.hstack([P, A.T])).sum(1).max(), np.abs(A).sum(1).max() + 1.0)
        tol = TOL[prec] * scale * max(1.0, *(np.max(np.abs(getattr(ref, v))) for v in ("x", "z", "y")))
        assert np.max(np.abs(res[name] - b)) <= tol, name
