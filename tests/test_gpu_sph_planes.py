"""Spherical reductions on grids that take one plane per block."""
import numpy as np
import pytest
import torch

import paper_2605_03563_amd as pg
from oracle import multipole as OM
from oracle import operators as OO

from .gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(16, 8, 16), (65, 10, 18), (64, 32, 80)])
def test_spherical_residual(dims):
    nr, nth, nph = dims
    say(f"spherical residual, one plane per block: {dims}")
    r, th, ph, ds = OM.sph_axes(nr, nth, nph)
    u, rho = np.random.default_rng(nph).standard_normal((2, nph, nth, nr + 2))
    plan = pg.Plan(pg.sph_grid(nr, nth, nph), pg.options("bicgstab", lmax=-1, max_iter=2))
    res = torch.zeros(u.shape, dtype=torch.float64, device="cuda:0")
    n2 = plan.residual(dev(rho), dev(u), res)
    ref = OO.sph_residual(u, rho, r, ds, th)
    assert np.max(np.abs(host(res)[:, :, 1:nr + 1] - ref)) < 1e-12 * np.max(np.abs(ref))
    assert abs(n2 / np.sum(ref ** 2) - 1.0) < 1e-12
    phi = dev(u)
    st = plan.solve(dev(rho), phi, tol=1e-30)
    left = np.linalg.norm(OO.sph_residual(host(phi), rho, r, ds, th))
    # the carried residual drifts by roundings of the start's
    assert abs(st.rel_residual * st.b_norm - left) < 1e-9 * np.linalg.norm(ref)
