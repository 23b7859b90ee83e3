"""Small grids queue one iteration ahead of the residual the host waits for:
a converged solve returns the iterate its iteration count names, bit for bit."""
import pytest
import torch

import paper_2605_03563_amd as pg
from paper_2605_03563_amd import _lib as L

from .gpu_util import dev, random_cart, say

pytestmark = pytest.mark.gpu

CASES = [("sor", 2, L.OMEGA_OPT, 1.0), ("sor", 2, L.OMEGA_CHEBYSHEV, 1.0), ("sor", 2, L.OMEGA_FIXED, 1.0),
         ("cg", 2, 0, 1.0), ("cg", 6, 0, 1.0), ("pcg", 2, 0, 1.0), ("pcg", 6, 0, 1.0)]


@pytest.mark.parametrize("check_every", [1, 2, 3, 5])
@pytest.mark.parametrize("method,order,mode,omega", CASES)
def test_converged_iterate(method, order, mode, omega, check_every):
    n, g = 24, 1 if order == 2 else 3
    say(f"iterate of {method} order {order} mode {mode} checked every {check_every}")
    phi, rho = random_cart(n, g, 5)

    def solve(tol, **kw):
        o = pg.options(method, order=order, lmax=-1, omega_mode=mode, omega=omega, **kw)
        x = dev(phi)
        r = pg.Plan(pg.cart_grid(n, ghost=g), o).solve(dev(rho), x, tol=tol, history=4000)
        return x, r

    x, r = solve(1e-7, check_every=check_every)
    assert r.converged and r.iterations % check_every == 0 and r.iterations > 10
    assert len(r.history) == 1 + r.iterations // check_every
    y, s = solve(1e-30, max_iter=r.iterations)
    assert not s.converged and s.iterations == r.iterations and s.rel_residual == r.rel_residual
    assert torch.equal(x, y)
    # the residual one check earlier had not met the tolerance
    assert r.history[-2] > 1e-7


@pytest.mark.parametrize("method", ["sor", "cg", "pcg", "mg", "mg_ir32"])
def test_plan_serves_many_solves(method):
    """Repeated solves of one plan with different tolerances, some converged at the start."""
    n = 24
    phi, rho = random_cart(n, 1, 6)
    plan = pg.Plan(pg.cart_grid(n), pg.options(method, lmax=-1, coarsest=6))
    first = None
    for tol in (1e-6, 1e-9, 1e-6, 1e-3):
        x = dev(phi)
        r = plan.solve(dev(rho), x, tol=tol)
        assert r.converged and r.rel_residual <= tol
        if tol == 1e-6:
            first = x if first is None else first
            assert torch.equal(x, first)
        again = plan.solve(dev(rho), x, tol=2 * tol)
        assert again.converged and again.iterations <= 1


def test_non_finite_density():
    n = 24
    phi, rho = random_cart(n, 1, 6)
    rho[5, 6, 7] = float("nan")
    for method in ("sor", "cg", "pcg", "mg"):
        plan = pg.Plan(pg.cart_grid(n), pg.options(method, lmax=-1, coarsest=6))
        with pytest.raises(pg.PoissonError):
            plan.solve(dev(rho), dev(phi), tol=1e-8)
        rho2 = random_cart(n, 1, 6)[1]
        assert plan.solve(dev(rho2), dev(phi), tol=1e-6).converged
