"""The large levels' four-colour pass of the 19-point star: sweeps against the
oracle at every residue of the row length, at the edges of its block sizes, and
on a zero guess (some colours taken as zero)."""
import numpy as np
import pytest

import paper_2605_03563_amd as pg
from oracle import smoothers as OS

from .gpu_util import dev, host, random_cart, rel_max, say

pytestmark = pytest.mark.gpu


# 96: smallest; 96..104: every residue of the unknowns' last column; 164 / 168:
# widest level of 256-lane blocks and narrowest of 512 (FP64); 205: 512 lanes,
# odd row count
@pytest.mark.parametrize("n", [96, 97, 98, 99, 100, 101, 102, 103, 104, 127, 164, 168, 205])
def test_sweep(n):
    say(f"four-colour sweep n {n}")
    phi, rho = random_cart(n, 3, n)
    plan = pg.Plan(pg.cart_grid(n, ghost=3), pg.options("cg", order=6, lmax=-1))
    x = dev(phi)
    plan.smooth(dev(rho), x, sweeps=1)
    ref = phi.copy()
    OS.smooth(ref, rho, n, 1.0 / n, 6, 3, forward=True)
    # values of order one after sums of 18 terms: a few ulp
    assert rel_max(host(x), ref) < 1e-13


# wide levels: 1024-lane blocks in FP64 (from 342 intervals) and 512 / 1024 in
# FP32; a refinement step of the mixed multigrid and an FP64 cycle contract the
# residual alike
@pytest.mark.parametrize("n,coarsest", [(104, 13), (112, 7), (352, 11), (448, 7)])
def test_cycles_agree(n, coarsest):
    say(f"19-point cycles n {n}")
    g = 3
    phi, rho = random_cart(n, g, 3)
    out = []
    for method in ("mg", "mg_ir32"):
        plan = pg.Plan(pg.cart_grid(n, ghost=g), pg.options(method, order=6, lmax=-1, coarsest=coarsest))
        x, d_rho = dev(phi), dev(rho)
        plan.vcycle(d_rho, x, cycles=1)
        res = plan.residual(d_rho, x, dev(np.zeros_like(phi)))
        out.append((host(x), res))
    # the mixed step's correction carries FP32 rounding (see test_gpu_small_levels)
    scale = np.max(np.abs(out[0][0] - phi))
    assert np.max(np.abs(out[0][0] - out[1][0])) < 5e-8 * n * n * scale
    assert abs(out[0][1] - out[1][1]) < 0.1 * out[0][1]
