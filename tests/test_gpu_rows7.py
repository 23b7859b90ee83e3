"""Cycles of the 7-point multigrid whose larger levels restrict their colour-0
residuals by rows: one and two compact columns per lane, full and partly
filled wavefronts, a level as wide as the kernel takes (its last lane reads a
ghost column), FP64 against the oracle's cycle and FP32 through the mixed
solve."""
import numpy as np
import pytest
import torch

import paper_2605_03563_amd as pg
from oracle import smoothers as OS
from tests.gpu_util import dev, host, rel_max, say

pytestmark = pytest.mark.gpu


def _problem(n):
    rng = np.random.default_rng(n)
    return rng.normal(size=(2, n + 1, n + 1, n + 1))


@pytest.mark.parametrize("n,coarsest", [(72, 9), (80, 5), (128, 8), (144, 9), (192, 6), (256, 8)])
def test_cycle_matches_oracle(n, coarsest):
    say(f"7-point rows: cycle n={n}")
    phi, rho = _problem(n)
    plan = pg.Plan(pg.cart_grid(n), pg.options("mg", order=2, lmax=-1, coarsest=coarsest))
    t = dev(phi)
    plan.vcycle(dev(rho), t, 1)
    ref = OS.vcycle(phi.copy(), rho, n, 1.0 / n, 2, 1, coarsest=coarsest)
    assert rel_max(host(t), ref) < 1e-12


@pytest.mark.parametrize("n,coarsest", [(72, 9), (128, 8), (160, 10), (256, 8)])
def test_mixed_solve_matches_fp64(n, coarsest):
    say(f"7-point rows: mixed solve n={n}")
    phi, rho = _problem(n)
    got = []
    for method in ("mg", "mg_ir32"):
        t = dev(phi)
        plan = pg.Plan(pg.cart_grid(n), pg.options(method, order=2, lmax=-1, coarsest=coarsest))
        st = plan.solve(dev(rho), t, tol=1e-11)
        assert st.converged and st.iterations <= 25
        got.append(host(t))
    # two iterates with residuals below 1e-11 of b's: within cond ~ n^2 / 2 of each other
    assert rel_max(got[1], got[0]) < 1e-11 * n * n
