"""The restricted residual leaves a mixed plan as it found it: the FP32
correction of later refinement steps keeps its zero boundary."""
import numpy as np
import pytest
import torch

import paper_2605_03563_amd as pg

from .gpu_util import dev, host, random_cart, say

pytestmark = pytest.mark.gpu


# finest levels swept by single passes (7-point above 64 intervals, the star),
# by the legs (64) and by one workgroup (16)
@pytest.mark.parametrize("order,n", [(2, 128), (2, 64), (2, 16), (6, 64), (6, 128)])
def test_mixed_plan_unchanged(order, n):
    say(f"restricted residual, then mixed solve: order {order} n {n}")
    g = 1 if order == 2 else 3
    phi, rho = random_cart(n, g, n + order)
    rho_d = dev(rho)
    out = []
    for first in (False, True):
        plan = pg.Plan(pg.cart_grid(n, ghost=g), pg.options("mg_ir32", order=order, lmax=-1, max_iter=30))
        if first:
            coarse = torch.zeros((n // 2 - 1) ** 3, dtype=torch.float64, device="cuda:0")
            plan.restrict_residual(rho_d, dev(phi), coarse)
        cycled = dev(phi)
        plan.vcycle(rho_d, cycled, cycles=2)
        solved = dev(phi)
        res = plan.solve(rho_d, solved, tol=1e-10)
        assert res.converged
        out.append((host(cycled), host(solved), res.iterations))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])
    assert out[0][2] == out[1][2]
