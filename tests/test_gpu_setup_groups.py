"""Set-up of more penalties than are factored together (their FP64 workspace stays within 1 GiB): the
matrices of every group are those of a handle with that penalty alone, so solves return its bits."""

import numpy as np
import pytest

from workloads import random_qp

pytestmark = pytest.mark.gpu


# n = m = 1500: about 55 MB of workspace per penalty in the single-instance engine (groups of 19), 127 MB
# in the batched one (groups of 8); penalties at the ends of the groups
@pytest.mark.parametrize("engine,prec,n_rho,indices", [
    ("single", "fp64", 24, (0, 18, 19, 23)), ("single", "fp32", 24, (18, 19, 23)),
    ("batch", "bf16x3", 17, (0, 7, 8, 15, 16)), ("batch", "fp32", 17, (7, 8, 16)),
])
def test_every_group_holds_its_penalties(engine, prec, n_rho, indices):
    import paper_2311_18056_amd as rq

    n = m = 1500
    P, q, A, l, u = random_qp(n, 0, m, seed=15)
    if engine == "batch":
        q, l, u = (np.tile(v, (3, 1)) for v in (q, l, u))
    # no penalty change: the only check is the last iteration
    kw = dict(precision=prec, engine=engine, eps_abs=0.0, eps_rel=0.0, max_iter=24)
    grid = np.logspace(-3, 3, n_rho)
    for j in indices:
        print(f"\n{engine} {prec}: penalty {j} of {n_rho}", flush=True)
        got = []
        for count in (n_rho, 1):
            # the start is the grid value nearest to rho0
            s = rq.Solver(P, q, A, l, u, n_rho=count, rho0=float(grid[j]), **kw)
            if count > 1:
                grid = np.asarray(s.rho_grid(), np.float64)
            s.solve()
            got.append(s.result())
            s.close()
        a, b = got
        assert np.all(np.asarray(a["iterations"]) == 24) and np.all(np.asarray(a["status"]) == rq.RQP_MAX_ITER)
        for name in ("x", "z", "y"):
            assert np.array_equal(a[name], b[name]), (j, name)
