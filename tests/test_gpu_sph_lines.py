"""Phi-line passes of the spherical preconditioner at the fixed splits of the
phi lines (2, 3, 4, 6, 8, 12 and 16 nodes in 16 segments, 2 in 8), at one that
takes the runtime split (80), with odd numbers of lines per colour, blocks
whose last lines are missing and tables per radius: one V(2,2) cycle against
the oracle's FP64 cycle."""
import numpy as np
import pytest
import torch

import paper_2605_03563_amd as pg
from oracle import multipole as OM
from oracle import sph_mg as SM
from oracle.radial import RadialMap
from tests.gpu_util import dev, host, rel_l2, say

pytestmark = pytest.mark.gpu
CYCLE_TOL = 1e-5  # a few roundings of 6e-8 per pass, where the lines are well conditioned


def _line_condition(nr, nth, nph, ds):
    """Condition number of the worst phi line (next to a pole): eigenvalues
    from D = 2 / ds^2 + 2 / dtheta^2 to D + 4 / (sin^2 dphi^2), on every level
    the same ratio.  An FP32 line solve is off by up to 2^-24 times it."""
    a = (nph / (2.0 * np.pi * np.sin(0.5 * np.pi / nth))) ** 2
    d = 2.0 / ds ** 2 + 2.0 * (nth / np.pi) ** 2
    return (d + 4.0 * a) / d


@pytest.mark.parametrize("pad", [False, True])
@pytest.mark.parametrize("dims", [(34, 8, 32), (12, 8, 96), (20, 8, 192), (12, 4, 256), (40, 8, 128), (10, 4, 80),
                                  (208, 64, 32), (6, 8, 16)])
def test_cycle_matches_oracle_at_every_split(dims, pad):
    nr, nth, nph = dims
    say(f"phi-line splits: cycle {dims} pad {pad}")
    if pad:
        grid = pg.sph_grid(nr, nth, nph, 0.2, 1.0, ext_in=nr // 5, ext_out=1, r_pad=0.1)
        lv = SM.level0(RadialMap(nr, 0.2, 1.0, ext_in=nr // 5, ext_out=1, r_pad=0.1), nr)
    else:
        grid = pg.sph_grid(nr, nth, nph)
        lv = OM.sph_axes(nr, nth, nph)[3]
    ds = RadialMap(nr, 0.2, 1.0, ext_in=nr // 5, ext_out=1, r_pad=0.1).ds if pad else lv
    tol = max(CYCLE_TOL, 2.0 ** -24 * _line_condition(nr, nth, nph, ds))
    plan = pg.Plan(grid, pg.options("bicgstab_mg32", lmax=-1))
    y = np.zeros((nph, nth, nr + 2))
    y[:, :, 1:nr + 1] = np.random.default_rng(sum(dims)).standard_normal((nph, nth, nr))
    yhat = torch.zeros(y.shape, dtype=torch.float64, device="cuda:0")
    for _ in range(2):  # the second call starts from the first one's workspace
        plan.precond(dev(y), yhat)
        err = rel_l2(host(yhat)[:, :, 1:nr + 1], SM.vcycle(y[:, :, 1:nr + 1], lv))
        say(f"  rel L2 {err:.2e} tol {tol:.2e}")
        assert err < tol


@pytest.mark.parametrize("pad", [False, True])
@pytest.mark.parametrize("dims,nu", [((16, 16, 8), (2, 2)), ((16, 12, 12), (2, 2)), ((18, 8, 16), (1, 3)),
                                     ((16, 8, 20), (2, 1)), ((16, 16, 24), (2, 2)), ((12, 8, 28), (2, 2)),
                                     ((32, 16, 32), (2, 2)), ((40, 12, 32), (3, 1)), ((64, 24, 32), (2, 2)), ((64, 8, 32), (2, 2))])
def test_small_levels_in_one_workgroup(dims, nu, pad):
    """Grids that are, or lead to, levels one workgroup runs: segments of 2 to
    8 nodes (odd ones restrict across segments), one and two smoothed levels,
    odd coarsest sizes, all threads busy, sweeps before and after that differ."""
    nr, nth, nph = dims
    say(f"small spherical levels: {dims} nu {nu} pad {pad}")
    args = (nr, 0.2, 1.0)
    ext = dict(ext_in=nr // 5, ext_out=1, r_pad=0.1)
    ds = RadialMap(*args, **ext).ds if pad else OM.sph_axes(nr, nth, nph)[3]
    lv = SM.level0(RadialMap(*args, **ext), nr) if pad else ds
    grid = pg.sph_grid(nr, nth, nph, 0.2, 1.0, **ext) if pad else pg.sph_grid(nr, nth, nph)
    plan = pg.Plan(grid, pg.options("bicgstab_mg32", lmax=-1, nu1=nu[0], nu2=nu[1]))
    tol = max(CYCLE_TOL, 2.0 ** -24 * _line_condition(nr, nth, nph, ds))
    y = np.zeros((nph, nth, nr + 2))
    y[:, :, 1:nr + 1] = np.random.default_rng(sum(dims)).standard_normal((nph, nth, nr))
    yhat = torch.zeros(y.shape, dtype=torch.float64, device="cuda:0")
    ref = SM.vcycle(y[:, :, 1:nr + 1], lv, nu1=nu[0], nu2=nu[1])
    for _ in range(2):
        plan.precond(dev(y), yhat)
        err = rel_l2(host(yhat)[:, :, 1:nr + 1], ref)
        say(f"  rel L2 {err:.2e} tol {tol:.2e}")
        assert err < tol


@pytest.mark.parametrize("method,dims", [("bicgstab", (70, 130, 66)), ("bicgstab", (70, 130, 94)),
                                         ("bicgstab", (70, 130, 250)), ("bicgstab_mg32", (136, 64, 96)),
                                         ("bicgstab_mg32", (144, 64, 192))])
def test_reductions_over_runs_of_planes(method, dims):
    """Grids whose reducing kernels take 2, 3, 4 and 8 planes per block, the last
    run shorter: residual and its norm, and the residual BiCGSTAB carries
    along (its dot products steer it) against that of the solution it returns."""
    from oracle import operators as OO
    nr, nth, nph = dims
    say(f"runs of planes: {method} {dims}")
    r, th, ph, ds = OM.sph_axes(nr, nth, nph)
    rng = np.random.default_rng(nph)
    u, rho = rng.standard_normal((2, nph, nth, nr + 2))
    plan = pg.Plan(pg.sph_grid(nr, nth, nph), pg.options(method, lmax=-1, max_iter=3))
    res = torch.zeros(u.shape, dtype=torch.float64, device="cuda:0")
    n2 = plan.residual(dev(rho), dev(u), res)
    ref = OO.sph_residual(u, rho, r, ds, th)
    assert np.max(np.abs(host(res)[:, :, 1:nr + 1] - ref)) < 1e-12 * np.max(np.abs(ref))
    assert abs(n2 / np.sum(ref ** 2) - 1.0) < 1e-12
    phi = dev(u)
    st = plan.solve(dev(rho), phi, tol=1e-30)
    left = np.linalg.norm(OO.sph_residual(host(phi), rho, r, ds, th))
    say(f"  {st.iterations} iterations, residual {left:.3e} after {np.linalg.norm(ref):.3e}")
    # the carried residual drifts by roundings of the start's
    assert abs(st.rel_residual * st.b_norm - left) < 1e-9 * np.linalg.norm(ref)
