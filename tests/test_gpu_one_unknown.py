"""Grids of two intervals, one unknown: every Cartesian method, both orders."""
import numpy as np
import pytest

import paper_2605_03563_amd as pg
from oracle import operators as OO

from .gpu_util import dev, host, random_cart, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,method", [(2, "sor"), (2, "cg"), (2, "pcg"), (2, "mg"), (2, "mg_ir32"), (6, "cg"),
                                          (6, "pcg"), (6, "mg"), (6, "mg_ir32")])
def test_solve(order, method):
    say(f"one unknown: {method} order {order}")
    g = 1 if order == 2 else 3
    phi, rho = random_cart(2, g, 4)
    plan = pg.Plan(pg.cart_grid(2, ghost=g), pg.options(method, order=order, lmax=-1, coarsest=2, max_iter=20))
    x = dev(phi)
    st = plan.solve(dev(rho), x, tol=1e-12)
    assert st.converged
    r = OO.residual(host(x), rho, 2, 0.5, order, g)
    assert abs(float(r[0, 0, 0])) < 1e-11 * st.b_norm
    out = rho.copy()
    t = dev(out)  # result in place of an input: the converting path
    n2 = plan.residual(t, dev(phi), t)
    ref = OO.residual(phi, rho, 2, 0.5, order, g)
    s = slice(g, g + 1)
    assert np.allclose(host(t)[s, s, s], ref, rtol=1e-13)
    assert n2 == pytest.approx(float(ref[0, 0, 0]) ** 2, rel=1e-12)
