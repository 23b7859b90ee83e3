"""Multigrid plans whose only level is the coarsest one: the exact solve takes
the potential's ghost values into account."""
import numpy as np
import pytest

import paper_2605_03563_amd as pg
from oracle import smoothers as OS

from .gpu_util import dev, host, random_cart, rel_max, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["mg", "mg_ir32"])
@pytest.mark.parametrize("order,n", [(2, 2), (2, 8), (2, 12), (6, 4), (6, 9)])
def test_cartesian(order, n, method):
    say(f"single level: {method} order {order} n {n}")
    g = 1 if order == 2 else 3
    phi, rho = random_cart(n, g, n)
    s = slice(g, g + n - 1)
    phi[s, s, s] = np.random.default_rng(n).normal(size=(n - 1,) * 3)
    plan = pg.Plan(pg.cart_grid(n, ghost=g), pg.options(method, order=order, lmax=-1, coarsest=n, max_iter=12))
    ref = OS.vcycle(phi.copy(), rho, n, 1.0 / n, order, g, coarsest=n)
    if method == "mg":
        x = dev(phi)
        plan.vcycle(dev(rho), x, cycles=1)
        assert rel_max(host(x), ref) < 1e-11
    x = dev(phi)
    st = plan.solve(dev(rho), x, tol=1e-12)
    assert st.converged and st.iterations <= (2 if method == "mg" else 4)
    # residual 1e-12 times the operator's condition, below 100 on these grids
    assert rel_max(host(x), ref) < 1e-10


@pytest.mark.parametrize("order,n,coarse_tol", [(2, 8, 0.0), (4, 9, 0.0), (6, 8, 0.0), (4, 8, 0.01)])
def test_spai(order, n, coarse_tol):
    say(f"single level: SPAI order {order} n {n} coarse_tol {coarse_tol}")
    g = 2 if order == 6 else 1
    phi, rho = random_cart(n, g, n)
    plan = pg.Plan(pg.cart_grid(n, ghost=g),
                   pg.options("mg_spai", order=order, lmax=-1, coarsest=n, max_iter=12, coarse_tol=coarse_tol))
    x = dev(phi)
    st = plan.solve(dev(rho), x, tol=1e-11)
    assert st.converged and st.iterations <= (2 if coarse_tol == 0.0 else 8)
    left = plan.residual(dev(rho), x, dev(np.zeros_like(phi))) ** 0.5
    assert left < 1.01e-11 * st.b_norm
