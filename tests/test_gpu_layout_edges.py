"""Layout conversions on both sides of their size rule (81 nodes per axis) and
with pitched rows."""
import numpy as np
import pytest
import torch

import paper_2605_03563_amd as pg

from .gpu_util import dev, host, random_cart, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n", [(2, 2), (2, 63), (2, 80), (2, 81), (6, 2), (6, 76), (6, 77)])
def test_round_trip(order, n):
    """No sweep: the unknowns come back bit for bit, the rest is left alone."""
    say(f"layout round trip: order {order} n {n}")
    g = 1 if order == 2 else 3
    m = n + 1 + 2 * (g - 1)
    plan = pg.Plan(pg.cart_grid(n, ghost=g, pitch_x=m + 3), pg.options("cg", order=order, lmax=-1))
    x = torch.randn(m, m, m + 3, dtype=torch.float64, device="cuda:0")
    rho = torch.randn_like(x)
    before = host(x).copy()
    plan.smooth(rho, x, sweeps=0)
    assert np.array_equal(host(x), before)


@pytest.mark.parametrize("n", [80, 88])
def test_single_precision(n):
    """Restricted residual of a mixed plan: Phi and rho converted to FP32."""
    say(f"layout in FP32: n {n}")
    phi, rho = random_cart(n, 1, n)
    out = []
    for method in ("mg", "mg_ir32"):
        plan = pg.Plan(pg.cart_grid(n), pg.options(method, lmax=-1, coarsest=10 if n == 80 else 11))
        coarse = torch.zeros((n // 2 - 1) ** 3, dtype=torch.float64, device="cuda:0")
        plan.restrict_residual(dev(rho), dev(phi), coarse)
        out.append(host(coarse))
    # FP32 rounds the inputs and the six-neighbour sums (relative 6e-8 each), weighted means keep it
    assert np.max(np.abs(out[0] - out[1])) < 2e-6 * np.max(np.abs(out[0]))
