"""The kernels that run a small multigrid level's leg, or all the coarsest
levels, in one launch: one cycle against the oracle's, at the sizes where their
tiles, slots and coarsest blocks end."""
import numpy as np
import pytest

import paper_2605_03563_amd as pg
from oracle import smoothers as OS

from .gpu_util import dev, host, random_cart, rel_max, say

pytestmark = pytest.mark.gpu

# (order, n, coarsest): levels of 2 and 3 coarse nodes, an even and an odd count
# of coarsest unknowns, the largest levels of each kernel size, blocks too many
# for LDS (coarsest 10), a coarsest level too large for one thread per row (12),
# and block rows of the legs that end inside the level
SIZES = [(2, 8, 2), (2, 16, 8), (2, 20, 5), (2, 24, 3), (2, 28, 7), (2, 36, 9), (2, 40, 10), (2, 44, 11), (2, 48, 12),
         (2, 64, 8), (2, 80, 5), (6, 16, 8), (6, 20, 5), (6, 24, 3), (6, 32, 8), (6, 36, 9),
         (6, 40, 10), (6, 56, 7)]


def _cycle(order, n, coarsest, nu1, nu2, method):
    g = 1 if order == 2 else 3
    phi, rho = random_cart(n, g, 7 * n + order)
    plan = pg.Plan(pg.cart_grid(n, ghost=g), pg.options(method, order=order, lmax=-1, coarsest=coarsest, nu1=nu1, nu2=nu2))
    t = dev(phi)
    plan.vcycle(dev(rho), t, cycles=1)
    return phi, rho, host(t)


@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1), (1, 2), (3, 1), (0, 2), (2, 0)])
@pytest.mark.parametrize("order,n,coarsest", SIZES)
def test_cycle(order, n, coarsest, nu1, nu2):
    say(f"cycle order {order} n {n} coarsest {coarsest} V({nu1},{nu2})")
    phi, rho, got = _cycle(order, n, coarsest, nu1, nu2, "mg")
    g = 1 if order == 2 else 3
    ref = OS.vcycle(phi.copy(), rho, n, 1.0 / n, order, g, nu1=nu1, nu2=nu2, coarsest=coarsest)
    assert rel_max(got, ref) < 1e-12


@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 1), (0, 2)])
@pytest.mark.parametrize("order,n,coarsest", SIZES)
def test_mixed_step(order, n, coarsest, nu1, nu2):
    """One refinement step: the FP32 cycle's correction, whose residuals carry
    rounding errors of eps 6 n^2 |e| that the coarse solves scale by about
    1 / (3 pi^2): 6e-8 n^2 / 5 of the correction, with a factor four."""
    say(f"mixed order {order} n {n} coarsest {coarsest} V({nu1},{nu2})")
    phi, rho, got = _cycle(order, n, coarsest, nu1, nu2, "mg_ir32")
    g = 1 if order == 2 else 3
    ref = OS.vcycle(phi.copy(), rho, n, 1.0 / n, order, g, nu1=nu1, nu2=nu2, coarsest=coarsest)
    scale = np.max(np.abs(ref - phi))
    assert np.max(np.abs(got - ref)) < max(5e-8 * n * n, 1e-5) * scale
