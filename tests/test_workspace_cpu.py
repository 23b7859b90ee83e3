"""A plan accepts the workspace that callers of its grid and options have passed
before: tables and flags that kernels keep there do not make it larger."""
import pytest

import paper_2605_03563_amd as pg

# method, intervals, order, coarsest, bytes: the scalars' flags (every plan) and
# the row table of the smallest coarsest levels (2, 3 and 4 intervals)
CART = [("sor", 32, 2, 8, 3320832), ("cg", 20, 6, 8, 5902592), ("pcg", 64, 2, 8, 36860672),
        ("mg", 8, 2, 2, 1369096), ("mg", 48, 2, 3, 6948608), ("mg", 64, 2, 4, 17501128), ("mg", 64, 2, 8, 18369416),
        ("mg_ir32", 16, 2, 2, 2099464), ("mg_ir32", 24, 6, 3, 6068992), ("mg_ir32", 40, 6, 5, 12570368),
        ("mg_spai", 32, 4, 8, 5157000), ("mg_spai32", 64, 2, 8, 17454472)]
SPH = [("bicgstab", (16, 8, 16), 1228800), ("sor", (16, 8, 16), 1232512), ("bicgstab_mg32", (32, 16, 32), 3105280),
       ("bicgstab_mg32", (64, 32, 64), 12641280)]


@pytest.mark.parametrize("method,n,order,coarsest,size", CART)
def test_cartesian(method, n, order, coarsest, size):
    ghost = 3 if order == 6 else 1
    got = pg.workspace_bytes(pg.cart_grid(n, ghost=ghost), pg.options(method, order=order, coarsest=coarsest))
    assert 0 < got <= size


@pytest.mark.parametrize("method,dims,size", SPH)
def test_spherical(method, dims, size):
    assert 0 < pg.workspace_bytes(pg.sph_grid(*dims), pg.options(method)) <= size
