"""Cartesian multipole moments and ghost values at every order the expansion
takes (each sums a different number of pairs per wavefront), on odd sizes with
one to three ghost layers, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2605_03563_amd as pg
from oracle import multipole as OM
from tests.gpu_util import dev, host, rel_max, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lmax", range(9))
@pytest.mark.parametrize("n,g", [(9, 1), (33, 1), (66, 3)])
def test_moments_and_ghosts_at_every_order(n, g, lmax):
    say(f"multipole n {n} g {g} lmax {lmax}")
    rng = np.random.default_rng(10 * n + lmax)
    m = n + 1 + 2 * (g - 1)
    rho = np.zeros((m, m, m))
    rho[g:-g, g:-g, g:-g] = rng.uniform(0.5, 1.5, size=(n - 1,) * 3)
    plan = pg.Plan(pg.cart_grid(n, ghost=g), pg.options("cg", order=6 if g == 3 else 2, lmax=lmax))
    phi = torch.zeros(rho.shape, dtype=torch.float64, device="cuda:0")
    q = np.array(plan.multipole_boundary(dev(rho), phi, lmax))
    ref_phi, ref_q = OM.cart_boundary(rho, n, g, lmax)
    assert rel_max(q, ref_q) < 1e-12
    mask = OM.cart_ghost_mask(n, g)
    got = host(phi)
    assert rel_max(got[mask], ref_phi[mask]) < 1e-12
    assert np.all(got[~mask] == 0.0)
