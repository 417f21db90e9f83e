"""The persistent kernel's layer-input words: a workgroup may overwrite a word only when every other
one has read it. CPU: a model of the protocol with the kernel's own rules for tags and halves
(``word_half`` and ``solve_span`` of layer_kernel.h, compiled for the host), one workgroup as late as
its dependences allow, through closed-loop steps of every small budget that end without a check. GPU: closed loops of odd
budgets against the FP64 oracle."""

import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from oracle import admm
from oracle.closed_loop import closed_loop
from workloads import random_mpc, x0_batch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2311_18056_amd", "csrc")

PROGRAM = r"""
#include "layer_kernel.h"
#include <cstdio>
// Steps of `budget` iterations without a check. The fast workgroup publishes a word as soon as it has
// gathered the one before it; the late one has published word k of a step but not yet gathered it. It
// still needs the fast workgroup's word k: lost if the next word published went to the same half.
int main() {
  for (int budget = 1; budget <= 40; ++budget) {
    uint32_t half[2] = {0, 0};  // tag of the fast workgroup's word in each half
    uint32_t tag = 1;
    uint32_t awaited = 0;  // the word that the late workgroup still polls for
    int awaited_half = 0;
    for (int step = 0; step < 5; ++step, tag += rqp::solve_span(budget))
      for (int k = 1; k <= budget; ++k) {
        half[rqp::word_half(tag, k)] = tag + k;
        if (awaited && half[awaited_half] != awaited) {
          std::printf("budget %d, step %d: word %d overwrites a word that is still read\n", budget, step, k);
          return 1;
        }
        awaited = tag + k;
        awaited_half = rqp::word_half(tag, k);
      }
  }
  std::printf("ok\n");
  return 0;
}
"""


def test_no_word_is_overwritten_while_it_is_read(tmp_path):
    src = tmp_path / "halves.cpp"
    src.write_text(PROGRAM)
    cc = shutil.which("g++") or "g++"
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = tmp_path / "halves"
    r = subprocess.run([cc, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", os.path.join(rocm, "include"),
                        str(src), "-o", str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


def test_the_kernel_places_its_words_by_that_rule():
    text = open(os.path.join(CSRC, "layer_impl.h")).read()
    uses = [ln.strip() for ln in text.splitlines() if re.search(r"\b(?:a\.)?xw \+ ", ln)]
    assert len(uses) == 3, uses  # first word of a segment, gather, update
    assert all("word_half(tag, " in ln for ln in uses), uses


@pytest.mark.gpu
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("fp32", 1e-4)])  # the closed loop's tolerances
@pytest.mark.parametrize("budget", [1, 3, 27])  # odd; 27: a check inside a step that ends without one
def test_closed_loop_of_an_odd_budget(prec, tol, budget):
    import torch

    import paper_2311_18056_amd as rq

    prob = random_mpc(15, 5, 40, seed=78)
    x0 = 8.0 * x0_batch(prob.nx, 1, 44)[0]
    steps = 30
    kw = dict(n_rho=1, eps_abs=0.0, eps_rel=0.0, max_iter=budget)
    q, l, u = prob.instance(x0)
    s = rq.Solver(prob.P, q, prob.A, l, u, precision=prec, engine="single", **kw)
    s.set_parametric(prob.F, prob.E, prob.lo, prob.hi)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")  # noqa: E731
    print(f"\nclosed loop: n + m = 400, {prec}, budget {budget}", flush=True)
    got = s.closed_loop(dev(x0), steps, dev(prob.A_dyn), dev(prob.B), prob.nu)
    got = {k: v.cpu().numpy() for k, v in got.items() if k != "_result"}
    s.close()
    xs, us, res = closed_loop(prob.P, prob.A, prob.F, prob.E, prob.lo, prob.hi, prob.A_dyn, prob.B, prob.nu, x0,
                              steps, admm.Settings(**kw))
    assert np.all(got["status"] == rq.RQP_MAX_ITER) and np.all(got["iterations"] == budget)
    for name, a, b in [("states", got["traj_x"], xs), ("controls", got["traj_u"], us)] + [
            (f"step {i} {v}", got[v][i], getattr(res[i], v)) for i in range(steps) for v in ("x", "z", "y")]:
        assert np.max(np.abs(a - b)) <= tol * max(np.max(np.abs(b)), 1.0), name
