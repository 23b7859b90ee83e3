"""Coarsest levels of 1, 8, 27 and 64 unknowns in the one-workgroup kernel: rows
with no table, rows of one thread, and sectors with fewer columns than there are
threads for a row."""
import pytest

from oracle import smoothers as OS

from .gpu_util import rel_max, say
from .test_gpu_small_levels import _cycle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,n,coarsest", [(2, 16, 2), (6, 16, 2), (2, 12, 3), (6, 12, 3), (2, 32, 4), (6, 16, 4),
                                              (2, 20, 5), (6, 40, 5)])
def test_cycle(order, n, coarsest):
    say(f"small coarsest level: order {order} n {n} coarsest {coarsest}")
    g = 1 if order == 2 else 3
    phi, rho, got = _cycle(order, n, coarsest, 2, 2, "mg")
    ref = OS.vcycle(phi.copy(), rho, n, 1.0 / n, order, g, nu1=2, nu2=2, coarsest=coarsest)
    assert rel_max(got, ref) < 1e-12
