"""BiCGstab where it leaves its regular course: <r0, A p> or omega vanishes exactly, the recursive residual meets the
tolerance before the true one does, and an error return, after which nothing may be left running on the stream.

On unit links with c_sw = 0 and periodic boundaries, A acts on the modes prod_d (-1)^x_d (d in a set of n directions) as
1/(2 kappa) - 4 + 2n, exactly also in floating point where that number and the amplitudes are small dyadic ones."""
import numpy as np
import pytest

from paper_1412_2629_amd import ddqcd, inputs
from tests.gpu_cases import Case, dev, host, rel

pytestmark = pytest.mark.gpu

L, BC = (4, 4, 4, 4), (1.0, 1.0, 1.0, 1.0)
V = 256


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def modes(counts):
    """A source whose 12 components hold counts[n] modes of n directions, amplitude 1."""
    i = np.arange(V)
    x = [i % 4, i // 4 % 4, i // 16 % 4, i // 64]
    f = np.zeros((V, 12), dtype=complex)
    k = 0
    for n, c in enumerate(counts):
        for _ in range(c):
            f[:, k] = np.prod([(-1.0) ** x[d] for d in range(n)], axis=0) if n else 1.0
            k += 1
    return f.reshape(V, 4, 3)


def context(kappa):
    ctx = ddqcd.Context(L, (2, 2, 2, 2), kappa, 0.0, BC)
    ctx.load_gauge(dev(inputs.unit_gauge(L)))
    return ctx


def recursion(apply, b, iterations):
    """BiCGstab from x = 0, restarted from the true residual where <r0, A p>, rho or omega vanishes."""
    x, r, restarts, it = np.zeros_like(b), b.copy(), 0, 0

    def begin():
        return r.copy(), np.zeros_like(b), np.zeros_like(b), 1.0, 1.0, 1.0

    r0, p, v, rho_old, alpha, omega = begin()
    while it < iterations:
        rho = np.vdot(r0, r)
        if rho == 0 or omega == 0:
            r = b - apply(x)
            r0, p, v, rho_old, alpha, omega = begin()
            restarts += 1
            continue
        beta = (rho / rho_old) * (alpha / omega)
        p = r + beta * (p - omega * v)
        v = apply(p)
        r0v = np.vdot(r0, v)
        if r0v == 0:
            r = b - apply(x)
            r0, p, v, rho_old, alpha, omega = begin()
            restarts += 1
            continue
        alpha = rho / r0v
        s = r - alpha * v
        t = apply(s)
        omega = np.vdot(t, s) / np.vdot(t, t).real
        x = x + alpha * p + omega * s
        r = s - omega * t
        rho_old = rho
        it += 1
    return x, r, restarts


@pytest.mark.parametrize("iterations", [1, 2, 3])
def test_restart_where_alpha_has_no_value(iterations, oracle):
    # 1/(2 kappa) = 2: eigenvalues -2, 0, 2, 4, 6; the first iteration has alpha = 1/2, omega = 1/8, beta = 1, and in the
    # second <r0, A p> = 0 while the restarted one has <r, A r> = -9
    U = inputs.unit_gauge(L)
    C = oracle.clover_field(L, U, 0.25, 0.0)
    b = modes((1, 2, 6, 2, 1))
    x, r, restarts = recursion(lambda f: oracle.apply_A(L, BC, U, C, f), b, iterations)
    assert restarts == (iterations > 1)
    ctx = context(0.25)
    got, info, st = ctx.solve_bicgstab(dev(b), max_iter=iterations, check=False)
    assert st == ddqcd.ERR_NOT_CONVERGED and info["iters"] == iterations and info["restarts"] == restarts
    # sums of 3072 products a few units in size, and a few such steps: 1e-12 is some thousand roundings
    assert rel(host(got), x) <= 1e-12
    assert abs(info["rel_residual"] - np.linalg.norm(r) / np.linalg.norm(b)) <= 1e-12


@pytest.mark.parametrize("kappa,counts", [(1 / 6, (1, 1, 0, 0, 0)),    # <b, A b> = 0 at once
                                          (1 / 6, (1, 0, 3, 0, 0))])   # omega = 0 after one step, then <r0, A p> = 0
def test_breakdown_is_an_error_and_the_context_goes_on(kappa, counts):
    b = dev(modes(counts))
    ctx = context(kappa)
    _, _, st = ctx.solve_bicgstab(b, check=False)
    assert st == ddqcd.ERR_NONFINITE
    good = dev(modes((3, 0, 1, 0, 2)))
    got, info, st = ctx.solve_bicgstab(good, max_iter=3, check=False)
    want, winfo, wst = context(kappa).solve_bicgstab(good, max_iter=3, check=False)
    assert st == wst and info["iters"] == winfo["iters"] and np.array_equal(host(got), host(want))


def test_recursive_residual_is_confirmed(oracle):
    # a tolerance that the recursion reaches and the true residual, with its roundings of A x, does not
    case = Case("8^4/4^4", (8, 8, 8, 8), (4, 4, 4, 4), 0.13, 1.5, 0.5, 601)
    b = case.source(33)
    ctx = case.context()
    ctx.set_solver(16, 1e-17, 64)
    x, info, st = ctx.solve_bicgstab(dev(b), max_iter=600, check=False)
    assert st == ddqcd.ERR_NOT_CONVERGED and info["iters"] == 600 and info["restarts"] > 0
    # the residual of the last restart's start: the roundings of A x, some tens of 1.1e-16
    assert rel(oracle.apply_A(case.L, (1.0, 1.0, 1.0, -1.0), case.U, case.C, host(x)), b) <= 1e-13


def test_nothing_runs_on_after_an_error():
    import torch
    # the last breakdown is found while the next direction, on a lattice where that takes half a millisecond, is queued
    big = (32, 32, 32, 32)
    n = 32 ** 4
    ctx = ddqcd.Context(big, (4, 4, 4, 4), 0.125, 0.0, BC)
    U = torch.eye(3, dtype=torch.complex128, device="cuda").expand(n, 4, 3, 3).contiguous()
    ctx.load_gauge(U)
    del U
    b = torch.ones(n, 4, 3, dtype=torch.complex128, device="cuda")   # A b = 0
    torch.cuda.synchronize()
    _, _, st = ctx.solve_bicgstab(b, check=False)
    idle = torch.cuda.current_stream().query()
    torch.cuda.synchronize()
    assert st == ddqcd.ERR_NONFINITE and idle
