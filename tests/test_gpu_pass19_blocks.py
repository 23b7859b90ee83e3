"""The four-colour pass at the edges of its block sizes.  A row of n intervals
has G = (n + 4) / 4 / c + 1 groups (rounded down; c = 2 columns in FP64, 4 in
FP32) and a block at least 12 G lanes: FP64 rows take 256 lanes up to 163
intervals, 512 up to 331 and 1024 up to 675, FP32 rows up to 331, 667 and
beyond."""
import pytest
import torch

import paper_2605_03563_amd as pg

from .gpu_util import say

pytestmark = pytest.mark.gpu


def _sweep(u, f, n):
    """One forward four-colour Gauss-Seidel sweep of the 19-point star (colour of
    a node: the sum of its indices modulo four), in place, in plain PyTorch."""
    g, e = 3, n - 1
    i = torch.arange(e, device=u.device) + 1
    colour = (i[:, None, None] + i[None, :, None] + i[None, None, :]) % 4
    weights = {1: 1.5, 2: -3.0 / 20.0, 3: 1.0 / 90.0}

    def window(dz, dy, dx):
        return u[g + dz:g + dz + e, g + dy:g + dy + e, g + dx:g + dx + e]

    for c in range(4):
        acc = f[g:g + e, g:g + e, g:g + e] / n ** 2
        for d, w in weights.items():
            for s in (-d, d):
                for off in ((s, 0, 0), (0, s, 0), (0, 0, s)):
                    acc.sub_(window(*off), alpha=w)
        acc.div_(-3.0 * 49.0 / 18.0)
        own = window(0, 0, 0)
        own.copy_(torch.where(colour == c, acc, own))
    return u


@pytest.mark.parametrize("n", [163, 164, 331, 332, 675])
def test_sweep(n):
    say(f"four-colour blocks: FP64 sweep n {n}")
    m = n + 5
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    u, f = (torch.randn(m, m, m, dtype=torch.float64, device="cuda:0", generator=gen) for _ in range(2))
    plan = pg.Plan(pg.cart_grid(n, ghost=3), pg.options("cg", order=6, lmax=-1))
    got = u.clone()
    plan.smooth(f, got, sweeps=1)
    ref = _sweep(u, f, n)
    # sums of 18 terms of order one: a few roundings of 1e-16
    assert float((got - ref).abs().max()) < 1e-13 * float(ref.abs().max())


@pytest.mark.parametrize("n,coarsest", [(320, 10), (352, 11), (640, 10), (704, 11)])
def test_single_precision_cycle(n, coarsest):
    """A mixed refinement step against the FP64 cycle, for a right-hand side that
    differs from node to node: a sweep then moves a node by about f h^2 / 8,
    some percent of the correction (0.1 h^1.5 f), and FP32 residuals err by 25
    roundings a level, 1e-5 of it, like f from node to node.  Nodes that a pass
    missed or formed from others stand out above 1e-4."""
    say(f"four-colour blocks: FP32 cycle n {n}")
    m = n + 5
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    f = torch.randn(m, m, m, dtype=torch.float64, device="cuda:0", generator=gen)
    out = []
    for method in ("mg", "mg_ir32"):
        plan = pg.Plan(pg.cart_grid(n, ghost=3),
                       pg.options(method, order=6, lmax=-1, coarsest=coarsest, nu1=2, nu2=1))
        x = torch.zeros_like(f)
        plan.vcycle(f, x, cycles=1)
        torch.cuda.synchronize()
        plan.close()
        del plan
        out.append(x)
    ref = out[0].abs().max()
    diff = float((out[0] - out[1]).abs().max() / ref)
    say(f"  {diff:.2e} of the correction; f h^2 / 8 is {float(f.abs().max() / n ** 2 / 8 / ref):.2e}")
    assert diff < 1e-4
