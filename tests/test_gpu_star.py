"""Residual, its norm and the operator on the caller's own arrays: sizes at the
edges of a wavefront's columns (58 star, 62 7-point), of a block's 16 rows and
of the runs of planes, pitched arrays, and results in place of an input (which
take the layout copies)."""
import numpy as np
import pytest
import torch

import paper_2605_03563_amd as pg
from oracle import operators as OO
from tests.gpu_util import dev, host, rel_max, say

pytestmark = pytest.mark.gpu
KTOL = 1e-12


@pytest.mark.parametrize("pad", [0, 5])
@pytest.mark.parametrize("n,order", [(8, 2), (8, 6), (62, 2), (63, 2), (64, 2), (58, 6), (59, 6), (60, 6), (17, 6),
                                     (18, 2), (117, 6), (126, 2)])
def test_residual_on_caller_arrays(n, order, pad):
    say(f"star residual n={n} order={order} pad={pad}")
    g = 3 if order == 6 else 1
    m = n + 1 + 2 * (g - 1)
    rng = np.random.default_rng(n + order)
    phi, rho = rng.standard_normal((2, m, m, m))
    s = slice(g, g + n - 1)

    def pitched(x):
        y = np.full((m, m, m + pad), np.nan)
        y[:, :, :m] = x
        return dev(y)

    plan = pg.Plan(pg.cart_grid(n, ghost=g, pitch_x=m + pad), pg.options("cg", order=order, lmax=-1))
    ref = OO.residual(phi, rho, n, 1.0 / n, order, g)
    zero = OO.residual(phi, np.zeros_like(rho), n, 1.0 / n, order, g)
    for where in ("apart", "rho", "phi"):
        d_phi, d_rho = pitched(phi), pitched(rho)
        res = {"apart": pitched(np.full((m, m, m), 7.0)), "rho": d_rho, "phi": d_phi}[where]
        n2 = plan.residual(d_rho, d_phi, res)
        assert rel_max(host(res)[s, s, s], ref) < KTOL, where
        assert n2 == pytest.approx(float(np.sum(ref * ref)), rel=1e-12)
        if where == "apart":  # only unknowns are written
            rest = host(res)[:, :, :m].copy()
            rest[s, s, s] = 7.0
            assert np.all(rest == 7.0)
            out = pitched(np.zeros((m, m, m)))
            plan.apply(d_phi, out)
            assert rel_max(host(out)[s, s, s], -zero) < KTOL
