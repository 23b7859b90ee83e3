"""7-point pass with two columns per lane where the last wavefront of a row is
partly filled: every residue of the row length, against the oracle, with ghost
values that differ from side to side."""
import pytest
import torch

import paper_2605_03563_amd as pg
from oracle import smoothers as OS

from .gpu_util import dev, host, random_cart, rel_max, say

pytestmark = pytest.mark.gpu


# two columns per lane from 256 intervals (128 columns, whole wavefronts); a full
# last pair has its right neighbours in a lane that owns no unknowns at 260, 288,
# 300 and 384
@pytest.mark.parametrize("n", [256, 257, 258, 259, 260, 288, 300, 301, 384])
def test_sweep(n):
    say(f"7-point sweep n {n}")
    phi, rho = random_cart(n, 1, n)
    plan = pg.Plan(pg.cart_grid(n), pg.options("cg", lmax=-1))
    x = dev(phi)
    plan.smooth(dev(rho), x, sweeps=1)
    ref = phi.copy()
    OS.smooth(ref, rho, n, 1.0 / n, 2, 1, forward=True)
    # sums of seven terms of order one: a few roundings
    assert rel_max(host(x), ref) < 1e-14


@pytest.mark.parametrize("n,coarsest,method", [(288, 9, "mg"), (320, 10, "mg"), (448, 7, "mg"), (576, 9, "mg"),
                                               (288, 9, "mg_ir32"), (576, 9, "mg_ir32"), (288, 9, "pcg")])
def test_solve_converges(n, coarsest, method):
    """Ghost values of an off-centre mass: the residual of what a solve returns
    meets its tolerance, by another kernel."""
    say(f"7-point solve {method} n {n}")
    plan = pg.Plan(pg.cart_grid(n), pg.options(method, lmax=4, coarsest=coarsest, max_iter=20 if method != "pcg" else 1500))
    ax = torch.arange(n + 1, dtype=torch.float64, device="cuda:0") / n - 0.4
    rho = torch.exp(-40.0 * (ax[:, None, None] ** 2 + ax[None, :, None] ** 2 + ax[None, None, :] ** 2))
    phi = torch.zeros_like(rho)
    st = plan.solve(rho, phi, tol=1e-7)
    assert st.converged
    left = plan.residual(rho, phi, torch.zeros_like(phi)) ** 0.5
    # FP64 cycles stop on the residual before their last smoothing
    assert left < 1.01e-7 * st.b_norm
