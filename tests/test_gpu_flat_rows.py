"""CG with lanes numbered over (compact column, row) pairs, and the norm of the
right-hand side with zero unknowns: rows that end inside, at and past a
block, few and many planes, ghosts that reach into every side.  Iterates and
norms against the oracle."""
import numpy as np
import pytest
import torch

import paper_2605_03563_amd as pg
from oracle import krylov as OK
from oracle import operators as OO
from tests.gpu_util import dev, host, rel_l2, say

pytestmark = pytest.mark.gpu
ITER_TOL = 1e-10     # FP64 iterates, reduction order differs


@pytest.mark.parametrize("method", ["cg", "pcg"])
@pytest.mark.parametrize("order,n", [(2, 9), (2, 31), (2, 129), (2, 150), (6, 8), (6, 67), (6, 130)])
def test_iterates_and_norm(order, n, method):
    say(f"flat rows: {method} order {order} n {n}")
    g = 1 if order == 2 else 3
    rng = np.random.default_rng(n + order)
    m = n + 1 + 2 * (g - 1)
    phi0, rho = rng.normal(size=(2, m, m, m))
    s = slice(g, g + n - 1)
    phi0[s, s, s] = 0.0
    hist = []
    OK.cg(phi0, rho, n, 1.0 / n, order, g, tol=0.0, max_iter=3, precondition=(method == "pcg"), history=hist)
    plan = pg.Plan(pg.cart_grid(n, ghost=g), pg.options(method, order=order, lmax=-1, max_iter=3))
    phi = dev(phi0)
    res = plan.solve(dev(rho), phi, tol=1e-30)
    assert res.iterations == 3
    assert rel_l2(host(phi)[s, s, s], hist[2]) < ITER_TOL
    b = OO.residual(phi0, rho, n, 1.0 / n, order, g)
    assert res.b_norm == pytest.approx(float(np.sqrt(np.sum(b * b))), rel=1e-12)
