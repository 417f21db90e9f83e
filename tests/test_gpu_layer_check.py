"""The persistent layer kernel on both sides of every change of its columns per lane, with row blocks in
registers, LDS and memory. Per iterate against the FP64 oracle with the penalty schedule replayed, and
the residuals that its checks publish against the same quantities formed on the CPU from the returned
x, z, y: the FP64 residual itself in FP64, the upper bound that certifies it in FP32."""

import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from oracle import admm
from workloads import random_qp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TOL = {"fp64": 1e-9, "fp32": 1e-4}  # the per-iterate tolerances of the FP64 and FP32 kernels

# columns per lane on both sides of each change of it (numbers of layer rows), up to the largest accepted
EDGES = {
    "fp32": {1: (129, 768), 2: (769, 2048), 3: (2049, 3072), 4: (3073, 4096), 5: (4097, 5120), 6: (5121, 6144),
             7: (6145, 7168), 8: (7169, 8192)},
    "fp64": {1: (129, 256), 2: (257, 2048), 3: (2049, 3072), 4: (3073, 4096), 5: (4097, 5120), 6: (5121, 6144),
             7: (6145, 7168), 8: (7169, 8192)},
}

PROGRAM = r"""
#include "layer_kernel.h"
#include <cstdio>
int main() {
  for (int L = 129; L <= rqp::kMaxLayerRows; ++L) {
    const int a = rqp::layer_col_lanes<float>(L), b = rqp::layer_col_lanes<double>(L);
    std::printf("%d %d %d\n", L, (L + a - 1) / a, (L + b - 1) / b);
  }
  return 0;
}
"""


def test_the_sizes_lie_at_the_edges_of_the_lane_rule(tmp_path):
    src, exe = tmp_path / "lanes.cpp", tmp_path / "lanes"
    src.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run([shutil.which("g++") or "g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I",
                        os.path.join(ROOT, "paper_2311_18056_amd", "csrc"), "-I", os.path.join(rocm, "include"),
                        str(src), "-o", str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    rows = [tuple(int(t) for t in ln.split()) for ln in r.stdout.splitlines()]
    for at, prec in ((1, "fp32"), (2, "fp64")):
        spans = {}
        for row in rows:
            lo, hi = spans.get(row[at], (row[0], row[0]))
            assert hi in (row[0], row[0] - 1)  # every number of columns holds one contiguous range
            spans[row[at]] = (lo, row[0])
        assert spans == EDGES[prec], prec


CASES = [(p, L, 0) for p in ("fp32", "fp64") for ends in EDGES[p].values() for L in ends]
CASES += [
    ("fp32", 700, 25), ("fp32", 2048, 40), ("fp32", 3073, 60),  # 28, 52 rows per workgroup: LDS, and memory
    ("fp64", 256, 5), ("fp64", 900, 20), ("fp64", 2049, 70),  # 52, 45, 30
]


def _published(prec, P, q, A, x, z, y):
    """(value, tolerance) of r_p and r_d as a check publishes them, in extended precision from the matrices
    and vectors as the handle holds them. With u = 2^-24 (an FP32 handle: P, A and q rounded to FP32, and
    the caller's own x, z, y): r = |residual| + kappa sum |a v| + 1.01 u |z or q| per row. The tolerance is
    that of the device's FP64 sums: at most 4 products per 256 columns and lane in a chain, then trees
    over 64 lanes and 16 waves and the row's own terms, each a rounding of 2^-53 of the sum of magnitudes."""
    n, m = P.shape[0], A.shape[0]
    ld = np.longdouble
    cast = (lambda a: a.astype(np.float32).astype(ld)) if prec == "fp32" else (lambda a: a.astype(ld))
    P, q, A = cast(P), cast(q), cast(A)
    x, z, y = x.astype(ld), z.astype(ld), y.astype(ld)
    kappa, ut = ld(0), ld(0)
    if prec == "fp32":
        kappa = 1.02 * (2 * ld(2) ** -24 + 2 * ld(n + m + 8) * ld(2) ** -53)
        ut = 1.01 * ld(2) ** -24
    sp = np.abs(A) @ np.abs(x)
    sd = np.abs(P) @ np.abs(x) + np.abs(A.T) @ np.abs(y)
    rp = np.abs(A @ x - z) + kappa * sp + ut * np.abs(z)
    rd = np.abs(P @ x + q + A.T @ y) + kappa * sd + ut * np.abs(q)
    ops = (4 * -(-(n + m) // 256) + 6 + 4 + 8) * ld(2) ** -53
    return (rp.max(), ops * (sp + np.abs(z)).max()), (rd.max(), ops * (sd + np.abs(q)).max())


@pytest.mark.gpu
@pytest.mark.parametrize("prec,L,grid", CASES)
def test_iterates_and_published_residuals(prec, L, grid):
    import paper_2311_18056_amd as rq

    n = 70 if L < 257 else 201  # no whole unit of the check's columns
    P, q, A, l, u = random_qp(n, 0, L - n, seed=L)
    cache = {}
    for max_iter in (25, 57):  # the first check alone; two checks and a ragged end
        print(f"\n{prec}: n = {n}, n + m = {L}, grid {grid}, {max_iter} iterations", flush=True)
        kw = dict(n_rho=2, rho_min=1e-2, rho_max=1.0, eps_abs=0.0, eps_rel=0.0, max_iter=max_iter)
        sol = rq.Solver(P, q, A, l, u, precision=prec, engine="single", **kw)
        if grid:
            sol.set_launch(grid)
        sol.solve()
        res = sol.result()
        sol.close()
        assert res["iterations"] == max_iter and res["status"] == rq.RQP_MAX_ITER
        ref = oracle.solve(P, q, A, l, u, admm.Settings(**kw), rho_replay=res["rho_hist"], cache=cache)
        for name in ("x", "z", "y"):
            a, b = res[name], getattr(ref, name)
            assert np.max(np.abs(a - b)) <= TOL[prec] * max(np.max(np.abs(b)), 1.0), name
        for name, (want, tol) in zip(("prim_res", "dual_res"), _published(prec, P, q, A, *(res[v] for v in "xzy"))):
            got = res[name][-1]
            assert abs(got - want) <= tol, (name, got, float(want), float(tol))
