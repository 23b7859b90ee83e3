"""The marching SPAI kernels (60-column wavefronts, runs of planes): cycles
against the oracle where tiles, rows and runs end inside the level."""
import pytest

from oracle import spai as SP

from .gpu_util import dev, host, rel_max, say
from .test_gpu_spai import _f, _nodes, _plan, _random

pytestmark = pytest.mark.gpu


# 55 unknowns per row: below one tile; 63, 71: into the second; 111, 143: two
# tiles and a rest; 12: coarse levels of 3 intervals
@pytest.mark.parametrize("nu1,nu2", [(3, 3), (1, 2), (0, 2), (2, 0)])
@pytest.mark.parametrize("order,n,coarsest", [(2, 12, 3), (4, 14, 7), (2, 56, 7), (6, 64, 8), (4, 72, 9), (2, 112, 7),
                                              (4, 144, 9)])
def test_cycle(order, n, coarsest, nu1, nu2):
    say(f"SPAI cycle order {order} n {n} coarsest {coarsest} V({nu1},{nu2})")
    phi, rho = _random(n, 3 * n + order, order)
    x = dev(phi)
    _plan(n, order, coarsest=coarsest, nu1=nu1, nu2=nu2).vcycle(dev(rho), x, 1)
    ref = _nodes(phi, n, order).copy()
    SP.vcycle(ref, SP.rhs_compact(_f(rho, n, order), n, order), n, SP.level_operators(order, n, coarsest),
              SP.COEFFS[order], nu1, nu2)
    assert rel_max(_nodes(host(x), n, order), ref) < 1e-12


# runs of 16 and of 32 planes with a remainder, ragged tiles and rows
@pytest.mark.parametrize("n", [160, 384])
def test_large_levels_agree_with_the_operator(n):
    """The solve's residual norm, formed by the marching kernel, is that of the
    residual operator."""
    say(f"SPAI residual norm n {n}")
    phi, rho = _random(n, n, 4)
    d_rho = dev(rho)
    plan = _plan(n, 4, coarsest=6 if n == 384 else 10, max_iter=1)
    x = dev(phi)
    r = plan.solve(d_rho, x, tol=1e-12)
    y = dev(phi)
    plan.vcycle(d_rho, y, 1)
    assert rel_max(host(x), host(y)) == 0.0
    norm = plan.residual(d_rho, x, dev(phi)) ** 0.5
    assert abs(r.rel_residual * r.b_norm / norm - 1.0) < 1e-11
