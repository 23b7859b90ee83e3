"""The host's side of the posts by which a solve's kernels report their sums: on
a HIP runtime without a GPU (hip_on_host.cpp) that runs no kernel and posts
the values that the test sets."""
import os
import subprocess
import sys
import textwrap

import pytest

from paper_2605_03563_amd import _lib as L

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

# Solver(method, grid, options): a plan on host memory with a stream of its own
# (so that iterations are recorded) or without
PRELUDE = """
import ctypes as C, sys
rt = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
import paper_2605_03563_amd as pg
from paper_2605_03563_amd import _lib as L
lib = L.load()
def knob(name, kind):
    return kind.in_dll(rt, name)
late, fail, turns = (knob("host_" + k, C.c_int) for k in ("late", "fail", "turns"))
b2, r2, later = (knob("host_" + k, C.c_double) for k in ("b2", "r2", "later"))
class Solver:
    def __init__(self, grid, opts, stream):
        self.grid, self.h = grid, C.c_void_p()
        n = lib.poisson_workspace_bytes(C.byref(grid), C.byref(opts))
        self.ws = C.create_string_buffer(n + 256)
        base = (C.addressof(self.ws) + 255) & ~255
        assert lib.poisson_plan(C.byref(self.h), C.byref(grid), C.byref(opts), base, n, stream) == L.OK
        self.x = C.create_string_buffer(8 * grid.pitch[1] * max(grid.n[2], grid.n[0] + 5))
    def __call__(self, tol=1e-8):
        st, p = L.Stats(), C.addressof(self.x)
        return lib.poisson_solve(self.h, p, p, C.byref(self.grid), tol, C.byref(st)), st
def cases():
    for stream in (None, C.c_void_p(8)):
        for method, n in (("mg", 16), ("mg", 128), ("mg_ir32", 32), ("sor", 16), ("cg", 16), ("pcg", 16), ("mg_spai", 16)):
            yield method, Solver(pg.cart_grid(n), pg.options(method, lmax=-1, max_iter=20), stream), stream
        for method in ("bicgstab", "bicgstab_mg32", "sor"):
            yield "spherical " + method, Solver(pg.sph_grid(16, 8, 16), pg.options(method, lmax=-1, max_iter=20), stream), stream
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rt") / "libhip_on_host.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
                    os.path.join(HERE, "hip_on_host.cpp"), "-o", out], check=True)
    return out


def _run(runtime, body):
    res = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), runtime], cwd=ROOT, text=True,
                         capture_output=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr


@pytest.mark.parametrize("late", [0, 1])
def test_residuals_reach_the_host(runtime, late):
    """Iterations end at max_iter, at once, or when the posted residual meets the
    tolerance; every solve of a plan reads its own posts."""
    _run(runtime, f"""
    late.value = {late}
    for name, solve, _ in cases():
        for b, r, want in ((4.0, 1.0, L.WARN_MAXITER), (9.0, 2.0 ** -70, L.OK), (1.0, 0.25, L.WARN_MAXITER)):
            b2.value, r2.value = b, r
            status, st = solve()
            assert status == want and st.b_norm == b ** 0.5 and st.rel_residual == r ** 0.5 / b ** 0.5, (name, b, status, st.b_norm)
            assert st.iterations == (0 if want == L.OK else 20), (name, st.iterations)
    """)


def test_post_left_by_a_failed_launch(runtime):
    """A launch that queues its work and reports an error leaves a post behind
    that the next solve must not take for its own."""
    _run(runtime, """
    late.value = 1
    for name, solve, stream in cases():
        if stream is None:
            continue
        b2.value, r2.value, fail.value = 4.0, 1.0, 1
        status, st = solve()
        if fail.value:  # methods that launch kernel by kernel
            fail.value = 0
            continue
        assert status == L.EHIP, name
        rt.hipStreamSynchronize(None)  # the post arrives
        b2.value = 9.0
        status, st = solve()
        assert status == L.WARN_MAXITER and st.b_norm == 3.0, (name, status, st.b_norm)
    """)


def test_nothing_runs_after_an_error(runtime):
    """A solve that gives up has waited for what it queued: the caller may free
    its arrays, the workspace and the plan."""
    _run(runtime, """
    for name, solve, _ in cases():
        b2.value, r2.value = 4.0, float("nan")
        assert solve()[0] == L.ENUMERIC, name
        assert rt.host_running() == 0, name
        r2.value, fail.value = 1.0, 1
        status, st = solve()
        assert status == (L.WARN_MAXITER if fail.value else L.EHIP), name
        assert rt.host_running() == 0, name
        fail.value = 0
    """)


def test_diverging_solve_has_ended(runtime):
    """The same where the residual stops being finite on the way."""
    _run(runtime, """
    for name, solve, _ in cases():
        b2.value, r2.value = 4.0, 1.0
        turns.value, later.value = 3, float("nan")
        assert solve()[0] == L.ENUMERIC, name
        assert rt.host_running() == 0, name
        turns.value = 0
    """)
