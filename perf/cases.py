"""Performance cases of the Poisson library: what a self-gravity code has it do.

Every case goes through the public Python entry points (``Plan.solve``, ``Plan.smooth``,
``Plan.residual``, ``Plan.multipole_boundary``, ``Server``).  The densities are the ones of the
library's workloads: Gaussian clumps (with or without a lognormal floor), a uniform sphere and a
perturbed singular isothermal sphere; 4 pi G = 1 on the unit box throughout.

``exact`` gives the same outputs by plain torch in 64 bits: the discrete solution by sine transforms
(7-point, compact stencils), by conjugate gradients around them (19-point star) or by a Fourier
transform with one tridiagonal solve per angular mode (log-spherical grid), under multipole ghost values
summed node by node.
"""
from __future__ import annotations

import math

import torch

import paper_2605_03563_amd as pg

DEV = "cuda:0"
F64 = torch.float64


# --------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest grid of the serving mix, from a cold start: launches and latency
        {"name": "mg_32", "kind": "solve", "method": "mg", "order": 2, "n": 32, "coarsest": 8, "lmax": 8, "tol": 1e-8,
         "rho": "clumps", "clumps": 8, "warm": False, "pad": 0},
        # a time step of a hydrodynamics code: mixed precision, the last step's potential as guess
        {"name": "mixed_128_warm", "kind": "solve", "method": "mg_ir32", "order": 2, "n": 128, "coarsest": 8,
         "lmax": 8, "tol": 1e-8, "rho": "clumps", "clumps": 16, "warm": True, "pad": 0},
        # the 255^3 clump workload, FP64 multigrid
        {"name": "mg_256", "kind": "solve", "method": "mg", "order": 2, "n": 256, "coarsest": 8, "lmax": 8,
         "tol": 1e-8, "rho": "clumps", "clumps": 16, "warm": False, "pad": 0},
        # the 512^3 recipe of the benchmark line: 19-point star, clumps on a lognormal floor
        {"name": "mg19_512", "kind": "solve", "method": "mg", "order": 6, "n": 512, "coarsest": 8, "lmax": 8,
         "tol": 1e-8, "rho": "floor", "clumps": 64, "warm": False, "pad": 0},
        # the same recipe at 256 intervals in mixed precision
        {"name": "mixed19_256", "kind": "solve", "method": "mg_ir32", "order": 6, "n": 256, "coarsest": 8, "lmax": 8,
         "tol": 1e-8, "rho": "floor", "clumps": 64, "warm": False, "pad": 0},
        # the paper's own multigrid in the shape of its table: 511^3 unknowns, seven coarse levels, V(3,3)
        {"name": "spai4_512", "kind": "solve", "method": "mg_spai", "order": 4, "n": 512, "coarsest": 4, "lmax": 8,
         "tol": 1e-8, "rho": "clumps", "clumps": 16, "warm": False, "pad": 0},
        # plain conjugate gradients on a grid that does not halve, rows padded by the caller
        {"name": "cg_150", "kind": "solve", "method": "cg", "order": 2, "n": 150, "coarsest": 8, "lmax": 8,
         "tol": 1e-6, "rho": "clumps", "clumps": 16, "warm": False, "pad": 5},
        # the uniform-sphere workload by red-black SOR: one small sweep and one test after another
        {"name": "sor_32", "kind": "solve", "method": "sor", "order": 2, "n": 32, "coarsest": 8, "lmax": 4,
         "tol": 1e-10, "rho": "sphere", "clumps": 0, "warm": False, "pad": 0},
        # the log-spherical isothermal sphere, BiCGSTAB with the FP32 multigrid preconditioner
        {"name": "sph_256x128x256", "kind": "sph", "nr": 256, "nth": 128, "nph": 256, "lmax": 8, "tol": 1e-8},
        # a burst of requests at the solve server, each stream warm from its last potential
        {"name": "serve_16", "kind": "serve", "n32": 6, "n64": 5, "n128": 3, "n256": 2, "slots": 8, "tol": 1e-8},
        # open-boundary values alone, for a code that iterates by itself
        {"name": "multipole_320", "kind": "multipole", "n": 320, "ghost": 3, "lmax": 8, "pad": 0},
        # the smoother and the residual as operators on a grid of no round size
        {"name": "smooth19_201", "kind": "smooth", "order": 6, "n": 201, "sweeps": 2, "pad": 2},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mg_size(rng, lo, hi):
    """A multigrid size coarsest * 2^L in [lo, hi]."""
    while True:
        want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        c = rng.choice((5, 6, 7, 8, 8, 8, 9, 10))
        n = c * 2 ** max(1, int(round(math.log2(want / c))))
        if lo <= n <= hi:
            return n, c


def draw(rng):
    kind = rng.choice(("mg", "mg", "mixed", "mixed", "mg19", "mixed19", "spai", "krylov", "sor", "sph", "serve",
                       "multipole", "smooth"))
    rho = {"rho": rng.choice(("clumps", "floor")), "clumps": rng.randint(1, 64), "warm": rng.random() < 0.4,
           "pad": rng.choice((0, 0, 0, 1, 6, 15)), "lmax": rng.choice((4, 6, 8, 8))}
    tol = 10.0 ** -rng.uniform(6.0, 9.0)
    if kind in ("mg", "mixed", "mg19", "mixed19"):
        n, c = _mg_size(rng, 24, 512 if kind == "mixed19" or not kind.endswith("19") else 448)
        return {"kind": "solve", "method": "mg" if kind.startswith("mg") else "mg_ir32",
                "order": 6 if kind.endswith("19") else 2, "n": n, "coarsest": c, "tol": tol, **rho}
    if kind == "spai":
        n, c = _mg_size(rng, 32, 512)
        return {"kind": "solve", "method": rng.choice(("mg_spai", "mg_spai", "mg_spai32")),
                "order": rng.choice((2, 4)), "n": n, "coarsest": c, "tol": tol, **rho}
    if kind == "krylov":
        return {"kind": "solve", "method": rng.choice(("cg", "pcg")), "order": rng.choice((2, 6)),
                "n": _log_int(rng, 20, 160), "coarsest": 8, "tol": max(tol, 1e-7), **rho}
    if kind == "sor":
        return {"kind": "solve", "method": "sor", "order": 2, "n": _log_int(rng, 16, 96), "coarsest": 8, "tol": tol,
                **rho}
    if kind == "sph":
        a, b = rng.choice(((8, 4), (8, 4), (7, 4), (9, 4), (10, 3), (6, 5))), 2 ** rng.choice((3, 4, 5))
        return {"kind": "sph", "nr": a[0] * b, "nth": a[1] * b, "nph": rng.choice((6, 8, 8, 8)) * b,
                "lmax": rng.choice((4, 8)), "tol": tol}
    if kind == "serve":
        return {"kind": "serve", "n32": rng.randint(1, 12), "n64": rng.randint(0, 8), "n128": rng.randint(0, 4),
                "n256": rng.randint(0, 2), "slots": rng.choice((2, 4, 8, 8)), "tol": tol}
    if kind == "multipole":
        return {"kind": "multipole", "n": _log_int(rng, 20, 512), "ghost": rng.choice((1, 3)),
                "lmax": rng.randint(2, 8), "pad": rho["pad"]}
    return {"kind": "smooth", "order": rng.choice((2, 6)), "n": _log_int(rng, 20, 320), "sweeps": rng.randint(1, 4),
            "pad": rho["pad"]}


def _ghost(case):
    return 3 if case["order"] == 6 else 1


def work(case):
    """Inputs read once and outputs written once; operations of the iterations such a case takes."""
    kind = case["kind"]
    if kind == "serve":
        sizes = [n for n, key in ((32, "n32"), (64, "n64"), (128, "n128"), (256, "n256")) for _ in range(case[key])]
        return {"bytes": sum(24.0 * (n + 1) ** 3 for n in sizes), "flops": sum(4e2 * n ** 3 for n in sizes)}
    if kind == "sph":
        nodes = float(case["nr"] * case["nth"] * case["nph"])
        return {"bytes": 16.0 * nodes, "flops": 2e3 * nodes}
    if kind == "multipole":
        n, m = case["n"], case["n"] + 2 * case["ghost"] - 1
        return {"bytes": 8.0 * (n - 1) ** 3 + 8.0 * (m ** 3 - (n - 1) ** 3), "flops": 17.0 * (n - 1) ** 3}
    nodes = float(case["n"] + 2 * _ghost(case) - 1) ** 3
    point = 37.0 if case["order"] == 6 else 13.0
    if kind == "smooth":
        return {"bytes": 32.0 * nodes, "flops": point * (case["sweeps"] + 1) * nodes}
    digits = -math.log10(case["tol"])
    steps = {"mg": 7.0 * digits, "mg_ir32": 7.0 * digits, "mg_spai": 5.0 * digits, "mg_spai32": 5.0 * digits,
             "cg": 0.3 * case["n"] * digits, "pcg": 0.3 * case["n"] * digits, "sor": 0.4 * case["n"] * digits}
    return {"bytes": (24.0 if case["warm"] else 16.0) * nodes, "flops": point * steps[case["method"]] * nodes}


# --------------------------------------------------------------------------- inputs
def _rng(seed):
    g = torch.Generator()
    g.manual_seed(0x5EED + 7919 * int(seed))
    return g


def _axis(n, ghost):
    return torch.arange(-(ghost - 1), n + ghost, dtype=F64, device=DEV) / n


def _draw_clumps(g, count):
    """Centres U[0.2, 0.8]^3, widths U[0.02, 0.08], masses lognormal(0, 0.5)."""
    c = 0.2 + 0.6 * torch.rand(count, 3, generator=g, dtype=F64)
    s = 0.02 + 0.06 * torch.rand(count, generator=g, dtype=F64)
    m = torch.exp(0.5 * torch.randn(count, generator=g, dtype=F64))
    return c.to(DEV), s.to(DEV), m.to(DEV)


def _clump_density(ax, clumps):
    c, s, m = clumps
    e = torch.exp(-(ax[None, None, :] - c[:, :, None]) ** 2 / (2 * s * s)[:, None, None])  # [clump][axis][node]
    amp = m * (2 * math.pi * s * s) ** -1.5
    k = ax.numel()
    zy = (amp[:, None] * e[:, 2])[:, :, None] * e[:, 1][:, None, :]
    return (zy.reshape(len(m), k * k).t().contiguous() @ e[:, 0].contiguous()).reshape(k, k, k)


def _clump_potential(ax, clumps):
    """The free-space potential of the clumps: a guess as good as a last time step's."""
    c, s, m = clumps
    phi = torch.zeros((ax.numel(),) * 3, dtype=F64, device=DEV)
    for i in range(len(m)):
        x, y, z = (ax - c[i, 0]) ** 2, (ax - c[i, 1]) ** 2, (ax - c[i, 2]) ** 2
        d = (z[:, None, None] + y[None, :, None] + x[None, None, :]).sqrt_().clamp_(min=1e-9)
        phi -= m[i] / (4 * math.pi) * torch.erf(d / (math.sqrt(2.0) * s[i])) / d
    return phi


def _floor(n, ghost, seed, mean):
    """Lognormal floor 0.05 mean exp(g - 1/2), g of unit variance with power |k|^-2."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 17)
    k = torch.fft.rfftn(torch.randn((n, n, n), generator=g, dtype=F64, device=DEV))
    f = torch.fft.fftfreq(n, d=1.0 / n, device=DEV, dtype=F64)
    fx = torch.fft.rfftfreq(n, d=1.0 / n, device=DEV, dtype=F64)
    k2 = f[:, None, None] ** 2 + f[None, :, None] ** 2 + fx[None, None, :] ** 2
    k *= torch.where((k2 >= 1.0) & (k2 <= (n / 2) ** 2), k2.clamp(min=1.0).rsqrt(), 0.0)
    del k2
    w = torch.fft.irfftn(k, s=(n, n, n))
    del k
    w -= w.mean()
    w /= w.std()
    i = (torch.arange(n + 2 * ghost - 1, device=DEV) - (ghost - 1)) % n
    return 0.05 * mean * torch.exp(w[i][:, i][:, :, i] - 0.5)


def _sphere(ax, g):
    c = 0.5 + 0.05 * (torch.rand(3, generator=g, dtype=F64).to(DEV) - 0.5)
    x, y, z = ((ax - c[d]) ** 2 for d in range(3))
    return (z[:, None, None] + y[None, :, None] + x[None, None, :] < 0.0625).to(F64)


def _padded(a, pad):
    if not pad:
        return a.contiguous()
    out = torch.zeros(a.shape[0], a.shape[1], a.shape[2] + pad, dtype=F64, device=DEV)
    out[:, :, :a.shape[2]] = a
    return out


def _cart_inputs(case, seed):
    """Density and initial potential on the nodes (ghost layers included), without row padding."""
    n, ghost, g = case["n"], _ghost(case), _rng(seed)
    ax = _axis(n, ghost)
    if case["rho"] == "sphere":
        return _sphere(ax, g), torch.zeros((ax.numel(),) * 3, dtype=F64, device=DEV)
    clumps = _draw_clumps(g, case["clumps"])
    if case["warm"]:  # the clumps a time step ago
        old = (clumps[0] + 0.002 * torch.randn(clumps[0].shape, generator=g, dtype=F64).to(DEV), clumps[1], clumps[2])
        phi = _clump_potential(ax, old)
    else:
        phi = torch.zeros((ax.numel(),) * 3, dtype=F64, device=DEV)
    rho = _clump_density(ax, clumps)
    if case["rho"] == "floor":
        rho += _floor(n, ghost, seed, float(clumps[2].sum()))
    return rho, phi


def _serve_inputs(case, seed):
    """Two densities for each stream of the burst: a request and its successor."""
    g, out = _rng(seed), []
    for n, key in ((256, "n256"), (128, "n128"), (64, "n64"), (32, "n32")):
        for _ in range(case[key]):
            c = _draw_clumps(g, int(torch.randint(1, 33, (1,), generator=g)))
            later = (c[0] + 0.002 * torch.randn(c[0].shape, generator=g, dtype=F64).to(DEV), c[1],
                     c[2] * torch.exp(0.02 * torch.randn(c[2].shape, generator=g, dtype=F64)).to(DEV))
            out.append((n, [_clump_density(_axis(n, 1), q) for q in (c, later)]))
    return out


R_MIN, R_MAX, R_OUT = 1e-3, 1.0, 0.8


def _sph_axes(case):
    ds = math.log(R_MAX / R_MIN) / (case["nr"] - 1)
    r = R_MIN * torch.exp(ds * torch.arange(-1, case["nr"] + 1, dtype=F64, device=DEV))
    th = (torch.arange(case["nth"], dtype=F64, device=DEV) + 0.5) * math.pi / case["nth"]
    ph = torch.arange(case["nph"], dtype=F64, device=DEV) * 2 * math.pi / case["nph"]
    return ds, r, th, ph


def _sph_density(case, seed):
    """rho = r^-2 (1 + a sin^2 theta cos 2(phi - phase)) inside R_OUT, zero in the radial ghosts."""
    _, r, th, ph = _sph_axes(case)
    u = torch.rand(2, generator=_rng(seed), dtype=F64)
    ang = 1.0 + (0.05 + 0.1 * float(u[0])) * torch.sin(th)[None, :] ** 2 * torch.cos(
        2.0 * (ph - math.pi * float(u[1])))[:, None]
    rad = torch.where(r < R_OUT, r ** -2, 0.0)
    rad[0] = 0.0
    rad[-1] = 0.0
    return (ang[:, :, None] * rad[None, None, :]).contiguous()


def _random_fields(case, seed):
    """A potential with its ghost values and a density for the operator cases: smooth fields plus noise."""
    n, ghost = case["n"], _ghost(case)
    ax, g = _axis(n, ghost), _rng(seed)
    clumps = _draw_clumps(g, 4)
    rho = _clump_density(ax, clumps)
    noise = torch.Generator(device=DEV)
    noise.manual_seed(int(seed) + 29)
    phi = _clump_potential(ax, clumps)
    phi += 0.01 * phi.std() * torch.randn(phi.shape, generator=noise, dtype=F64, device=DEV)
    return rho, phi


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        n, ghost = case["n"], _ghost(case)
        rho, phi = (_padded(a, case["pad"]) for a in _cart_inputs(case, seed))
        m = n + 2 * ghost - 1
        plan = pg.Plan(pg.cart_grid(n, ghost, pitch_x=m + case["pad"]),
                       pg.options(case["method"], case["order"], lmax=case["lmax"], coarsest=case["coarsest"]), DEV)
        return {"case": case, "plan": plan, "rho": rho, "guess": phi if case["warm"] else None,
                "phi": torch.zeros_like(phi)}
    if kind == "sph":
        plan = pg.Plan(pg.sph_grid(case["nr"], case["nth"], case["nph"], R_MIN, R_MAX),
                       pg.options("bicgstab_mg32", lmax=case["lmax"], point_mass=4 * math.pi * R_MIN), DEV)
        rho = _sph_density(case, seed)
        return {"case": case, "plan": plan, "rho": rho, "guess": None, "phi": torch.zeros_like(rho)}
    if kind == "serve":
        burst = _serve_inputs(case, seed)
        need = sum(80 * (n + 20) ** 3 for n, _ in burst) + (1 << 28)
        srv = pg.Server(need, max_slots=case["slots"], mixed=True, lmax=8, tol=case["tol"], device=DEV)
        for n in sorted({n for n, _ in burst}):
            srv.reserve(n, min(case["slots"], sum(k == n for k, _ in burst)))
        return {"case": case, "server": srv, "burst": burst, "turn": 0,
                "phi": [torch.zeros_like(r[0]) for _, r in burst]}
    if kind == "multipole":
        n, ghost, g = case["n"], case["ghost"], _rng(seed)
        rho = _padded(_clump_density(_axis(n, ghost), _draw_clumps(g, 16)), case["pad"])
        grid = pg.cart_grid(n, ghost, pitch_x=n + 2 * ghost - 1 + case["pad"])
        plan = pg.Plan(grid, pg.options("cg", 6 if ghost == 3 else 2), DEV)
        return {"case": case, "plan": plan, "rho": rho, "phi": torch.zeros_like(rho)}
    rho, phi = (_padded(a, case["pad"]) for a in _random_fields(case, seed))
    n, ghost = case["n"], _ghost(case)
    plan = pg.Plan(pg.cart_grid(n, ghost, pitch_x=n + 2 * ghost - 1 + case["pad"]),
                   pg.options("cg", case["order"], lmax=-1), DEV)
    return {"case": case, "plan": plan, "rho": rho, "guess": phi, "phi": phi.clone(), "res": torch.zeros_like(phi)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("solve", "sph"):
        phi = state["phi"]
        if state["guess"] is None:
            phi.zero_()
        else:
            phi.copy_(state["guess"])
        res = state["plan"].solve(state["rho"], phi, tol=case["tol"])
        return {"phi": phi, "iterations": res.iterations}
    if kind == "serve":
        srv, turn = state["server"], state["turn"] % 2
        state["turn"] += 1
        tickets = [srv.submit(i, n, rho[turn], state["phi"][i]) for i, (n, rho) in enumerate(state["burst"])]
        for t in tickets:
            srv.wait(t)
        return {"phi": state["phi"], "iterations": torch.tensor([srv.poll(t)[0].iterations for t in tickets])}
    if kind == "multipole":
        q = state["plan"].multipole_boundary(state["rho"], state["phi"], case["lmax"])
        return {"phi": state["phi"], "q": torch.tensor(q, dtype=F64)}
    state["phi"].copy_(state["guess"])
    state["plan"].smooth(state["rho"], state["phi"], case["sweeps"])
    state["plan"].residual(state["rho"], state["phi"], state["res"])
    return {"phi": state["phi"], "res": state["res"]}


# --------------------------------------------------------------------------- exact results, plain torch
def _solid(x, y, z, lmax):
    """Real regular solid harmonics sqrt(4 pi / (2l + 1)) r^l Y_lm as {(l, m): values}, one degree at a time."""
    r2 = x * x + y * y + z * z
    c, s = torch.ones_like(x), torch.zeros_like(x)
    for m in range(lmax + 1):
        if m:
            c, s = x * c - y * s, x * s + y * c
        lower, p = None, torch.full_like(x, math.prod(range(1, 2 * m, 2)))
        for l in range(m, lmax + 1):
            if l > m:
                q = (2 * l - 1) * z * p
                if l > m + 1:
                    q -= (l + m - 1) * r2 * lower
                lower, p = p, q / (l - m)
            a = math.sqrt((2.0 if m else 1.0) * math.factorial(l - m) / math.factorial(l + m))
            yield l, m, a * p * c
            if m:
                yield l, -m, a * p * s


def _cart_boundary(rho, n, ghost, lmax):
    """Multipole ghost values (the unknowns zero) and the moments."""
    ax = _axis(n, ghost)
    m, inner = ax.numel(), slice(ghost, ghost + n - 1)
    x = ax - 0.5
    r = torch.zeros((m, m, m), dtype=torch.bool, device=DEV)
    r[inner, inner, inner] = True
    q = torch.zeros((lmax + 1) ** 2, dtype=F64, device=DEV)
    w = rho[inner, inner, inner] / n ** 3
    xi, step = x[inner], 64
    for k in range(0, n - 1, step):
        z = xi[k:k + step]
        shape = (z.numel(), n - 1, n - 1)
        grid = (xi[None, None, :].expand(shape), xi[None, :, None].expand(shape), z[:, None, None].expand(shape))
        for l, mm, v in _solid(*grid, lmax):
            q[l * l + l + mm] += (w[k:k + step] * v).sum()
    kk, jj, ii = torch.nonzero(~r, as_tuple=True)
    gx, gy, gz = x[ii], x[jj], x[kk]
    d = (gx * gx + gy * gy + gz * gz).sqrt()
    val = torch.zeros_like(d)
    for l, mm, v in _solid(gx, gy, gz, lmax):
        val -= q[l * l + l + mm] * v / d ** (2 * l + 1)
    phi = torch.zeros((m, m, m), dtype=F64, device=DEV)
    phi[kk, jj, ii] = val / (4 * math.pi)
    return phi, q


STAR6 = (-49.0 / 18.0, 1.5, -0.15, 1.0 / 90.0)


def _apply(phi, n, ghost, order):
    """L phi at the unknowns (order 2, 6: 7-point and 19-point star)."""
    lo, e = ghost, n - 1
    c = slice(lo, lo + e)
    w = STAR6 if order == 6 else (-2.0, 1.0)
    out = 3 * w[0] * phi[c, c, c]
    for d in range(1, len(w)):
        up, dn = slice(lo + d, lo + d + e), slice(lo - d, lo - d + e)
        for a in ((up, c, c), (dn, c, c), (c, up, c), (c, dn, c), (c, c, up), (c, c, dn)):
            out += w[d] * phi[a]
    return out.mul_(float(n) ** 2)


def _compact4(u, lo, e):
    """Sums over the faces and edges around each unknown."""
    c, up, dn = slice(lo, lo + e), slice(lo + 1, lo + 1 + e), slice(lo - 1, lo - 1 + e)
    faces = u[up, c, c] + u[dn, c, c] + u[c, up, c] + u[c, dn, c] + u[c, c, up] + u[c, c, dn]
    edges = sum(u[a, b, c] + u[a, c, b] + u[c, a, b] for a in (up, dn) for b in (up, dn))
    return faces, edges


class _Sine:
    """Sine transforms along all axes and the symbols of the operators they diagonalise."""

    def __init__(self, n):
        k = torch.arange(1, n, dtype=F64, device=DEV)
        j = torch.arange(1, n, device=DEV)
        self.n = n
        self.s = math.sqrt(2.0 / n) * torch.sin(math.pi / n * ((j[:, None] * j[None, :]) % (2 * n)).to(F64))
        self.c = 2 * torch.cos(math.pi * k / n)
        c = self.c
        self.faces = c[:, None, None] + c[None, :, None] + c[None, None, :]

    def apply(self, a):
        e = self.n - 1
        for _ in range(3):  # one axis at a time, the last becoming the first
            a = (self.s @ a.reshape(e, e * e)).t().contiguous().reshape(e, e, e)
        return a

    def solve7(self, b):
        return self.apply(self.apply(b) / ((self.faces - 6.0) * float(self.n) ** 2))

    def solve_compact4(self, b):
        c = self.c
        edges = c[:, None, None] * c[None, :, None] + c[:, None, None] * c[None, None, :] + c[None, :, None] * c
        return self.apply(self.apply(b) / ((-24.0 + 2.0 * self.faces + edges) * (float(self.n) ** 2 / 6.0)))


def _exact_cart(rho, n, ghost, lmax, order, compact):
    """The discrete solution on all nodes."""
    phi, _ = _cart_boundary(rho, n, ghost, lmax)
    c, sine = slice(ghost, ghost + n - 1), _Sine(n)
    if compact and order == 4:
        fr, _ = _compact4(rho, ghost, n - 1)
        fb, eb = _compact4(phi, ghost, n - 1)
        u = sine.solve_compact4((6.0 * rho[c, c, c] + fr) / 12.0 - (2.0 * fb + eb) * (float(n) ** 2 / 6.0))
    elif order == 2:
        u = sine.solve7(rho[c, c, c] - _apply(phi, n, ghost, 2))
    else:
        b = rho[c, c, c] - _apply(phi, n, ghost, 6)
        u, wide = torch.zeros_like(b), torch.zeros_like(phi)
        r, bb = b.clone(), float(b.square().sum())
        z = sine.solve7(r)
        p, rz = z.clone(), float((r * z).sum())
        for _ in range(60):
            wide[c, c, c] = p
            q = _apply(wide, n, ghost, 6)
            a = rz / float((p * q).sum())
            u += a * p
            r -= a * q
            if float(r.square().sum()) <= 1e-26 * bb:
                break
            z = sine.solve7(r)
            rz, old = float((r * z).sum()), rz
            p = z + (rz / old) * p
    phi[c, c, c] = u
    return phi


def _mix(a, b):
    """Batched product of a real matrix and a complex one."""
    return torch.complex(torch.bmm(a, b.real.contiguous()), torch.bmm(a, b.imag.contiguous()))


def _exact_sph(case, seed):
    """Fourier modes in longitude, eigenvectors in colatitude, a tridiagonal solve in radius for each pair."""
    ds, r, th, ph = _sph_axes(case)
    nr, nth, nph, lmax = case["nr"], case["nth"], case["nph"], case["lmax"]
    rho, pm = _sph_density(case, seed), 4 * math.pi * R_MIN
    dth, dph = math.pi / nth, 2 * math.pi / nph
    st, ct = torch.sin(th), torch.cos(th)
    x, y, z = st[None, :] * torch.cos(ph)[:, None], st[None, :] * torch.sin(ph)[:, None], ct[None, :].expand(nph, nth)
    w = rho[:, :, 1:-1] * (r[1:-1] ** 3 * ds * dth * dph) * st[None, :, None]
    inner, outer = torch.zeros(nph, nth, dtype=F64, device=DEV), torch.zeros(nph, nth, dtype=F64, device=DEV)
    inner -= pm / float(r[0])
    for l, m, v in _solid(x.contiguous(), y.contiguous(), z.contiguous(), lmax):
        ray = (w * v[:, :, None]).sum((0, 1))
        q, qbar = float((ray * r[1:-1] ** l).sum()), float((ray * r[1:-1] ** (-l - 1)).sum())
        if l == 0:
            q += pm
        outer -= q * v * float(r[-1]) ** (-l - 1)
        inner -= qbar * v * float(r[0]) ** l
    inner /= 4 * math.pi
    outer /= 4 * math.pi
    cl, cr = ds ** -2 - 0.5 / ds, ds ** -2 + 0.5 / ds
    b = rho[:, :, 1:-1] * r[1:-1] ** 2
    b[:, :, 0] -= cl * inner
    b[:, :, -1] -= cr * outer
    bm = torch.fft.rfft(b, dim=0)
    tl = dth ** -2 - 0.5 * (ct / st) / dth
    tr = dth ** -2 + 0.5 * (ct / st) / dth
    scale = torch.ones(nth, dtype=F64, device=DEV)
    for j in range(1, nth):
        scale[j] = scale[j - 1] * torch.sqrt(tl[j] / tr[j - 1])
    off = torch.sqrt(tr[:-1] * tl[1:])
    modes = torch.arange(nph // 2 + 1, dtype=F64, device=DEV)
    mats = torch.zeros(nph // 2 + 1, nth, nth, dtype=F64, device=DEV)
    lam = 2.0 * (torch.cos(modes * dph) - 1.0) / dph ** 2
    i = torch.arange(nth, device=DEV)
    mats[:, i, i] = -2.0 * dth ** -2 + lam[:, None] / (st * st)
    sign = 1.0 - 2.0 * (modes % 2)
    mats[:, 0, 0] += sign * tl[0]
    mats[:, -1, -1] += sign * tr[-1]
    mats[:, i[:-1], i[1:]] = off
    mats[:, i[1:], i[:-1]] = off
    ev, vec = torch.linalg.eigh(mats.cpu())
    ev, vec = ev.to(DEV), vec.to(DEV)
    g = _mix(vec.transpose(1, 2).contiguous(), bm / scale[None, :, None]).permute(2, 0, 1).contiguous()
    diag = ev - (cl + cr)
    cp, gp = torch.empty(nr, *ev.shape, dtype=F64, device=DEV), torch.empty_like(g)
    cp[0], gp[0] = cr / diag, g[0] / diag
    for k in range(1, nr):
        den = diag - cl * cp[k - 1]
        cp[k], gp[k] = cr / den, (g[k] - cl * gp[k - 1]) / den
    for k in range(nr - 2, -1, -1):
        gp[k] -= cp[k] * gp[k + 1]
    out = _mix(vec, gp.permute(1, 2, 0)) * scale[None, :, None]
    phi = torch.zeros(nph, nth, nr + 2, dtype=F64, device=DEV)
    phi[:, :, 1:-1] = torch.fft.irfft(out, n=nph, dim=0)
    phi[:, :, 0], phi[:, :, -1] = inner, outer
    return phi


def _exact_smooth(case, seed):
    rho, phi = _random_fields(case, seed)
    n, ghost, order = case["n"], _ghost(case), case["order"]
    c, colours = slice(ghost, ghost + n - 1), 4 if order == 6 else 2
    k = torch.arange(1, n, device=DEV)
    colour = (k[:, None, None] + k[None, :, None] + k[None, None, :]) % colours
    diag = 3.0 * (STAR6[0] if order == 6 else -2.0) * float(n) ** 2
    b = rho[c, c, c]
    for _ in range(case["sweeps"]):
        for q in range(colours):
            u = phi[c, c, c]
            phi[c, c, c] = torch.where(colour == q, u + (b - _apply(phi, n, ghost, order)) / diag, u)
    res = torch.zeros_like(phi)
    res[c, c, c] = b - _apply(phi, n, ghost, order)
    return {"phi": _padded(phi, case["pad"]), "res": _padded(res, case["pad"])}


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        rho, _ = _cart_inputs(case, seed)
        phi = _exact_cart(rho, case["n"], _ghost(case), case["lmax"], case["order"], case["method"].startswith("mg_spai"))
        return {"phi": _padded(phi, case["pad"]), "iterations": None}
    if kind == "sph":
        return {"phi": _exact_sph(case, seed), "iterations": None}
    if kind == "serve":
        return {"phi": [_exact_cart(rho[0], n, 1, 8, 2, False) for n, rho in _serve_inputs(case, seed)],
                "iterations": None}
    if kind == "multipole":
        n, ghost = case["n"], case["ghost"]
        rho = _clump_density(_axis(n, ghost), _draw_clumps(_rng(seed), 16))
        phi, q = _cart_boundary(rho, n, ghost, case["lmax"])
        return {"phi": _padded(phi, case["pad"]), "q": q}
    return _exact_smooth(case, seed)
