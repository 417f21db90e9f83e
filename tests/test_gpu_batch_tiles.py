"""The batched kernel's 64-row shape where it goes in 32-row tiles: K loops shorter than the ring of
stages, ragged rows and instances, and batches on both sides of the number of tiles that decides it.
Per iterate against the FP64 oracle with the penalty schedule replayed."""

import numpy as np
import pytest

import oracle
from oracle import admm
from workloads import random_qp

TOL = {"fp32": 1e-4, "bf16x3": 5e-3}  # the batched engine's per-iterate tolerances


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("n,m,B", [
    (12, 8, 5), (20, 13, 130), (100, 61, 200),  # 1, 2 and 6 K stages
    (448, 448, 1100), (470, 460, 1100),  # 9 M tiles x 28 = 252 tiles of 32 rows, x 30 = 270
])
def test_small_row_tiles(prec, n, m, B):
    import paper_2311_18056_amd as rq

    P, q, A, l, u = random_qp(n, 0, m, seed=n)
    rng = np.random.default_rng(m)
    qs = q + 0.3 * rng.standard_normal((B, n))
    sol = rq.Solver(P, qs, A, np.tile(l, (B, 1)), np.tile(u, (B, 1)), precision=prec, engine="batch", n_rho=8,
                    eps_abs=0.0, eps_rel=0.0, max_iter=60)
    sol.set_tile(64)
    sol.solve()
    res = sol.result()
    sol.close()
    s = admm.Settings(n_rho=8, eps_abs=0.0, eps_rel=0.0, max_iter=60)
    assert (res["iterations"] == 60).all() and (res["status"] == rq.RQP_MAX_ITER).all()
    cache = {}
    for b in (0, B // 2, B - 1):
        ref = oracle.solve(P, qs[b], A, l, u, s, rho_replay=res["rho_hist"][b][:3].tolist(), cache=cache)
        for name in ("x", "z", "y"):
            a, r = res[name][b], getattr(ref, name)
            assert np.max(np.abs(a - r)) <= TOL[prec] * max(np.max(np.abs(r)), 1.0), (name, b)
