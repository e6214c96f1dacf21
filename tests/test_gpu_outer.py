"""The outer solvers' linear algebra, whose scalars stay on the device within a step: more systems than a launch holds
(16) with the bits of each alone, a Gram-Schmidt pass that has to be repeated, and BiCGstab step by step, against the
same recursions in numpy on the library's operator and preconditioner."""
import numpy as np
import pytest

from tests.gpu_cases import BC, Case, dev, host, rel

pytestmark = pytest.mark.gpu

CASE = Case("8^4/4^4", (8, 8, 8, 8), (4, 4, 4, 4), 0.13, 1.5, 0.5, 601)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("nrhs", [2, 16, 17])
def test_systems_of_a_launch(nrhs):
    ctx = CASE.context()
    ctx.set_sap(2, 3, "f32")
    ctx.set_solver(6, 1e-9, 40)
    f = dev(np.stack([CASE.source(30 + k) for k in range(nrhs)]))
    x, info, st = ctx.solve(f)
    assert st == 0
    for k in sorted({0, nrhs // 2, nrhs - 1}):
        xk, ik, sk = ctx.solve(f[k].contiguous())
        assert sk == 0 and np.array_equal(host(xk), host(x[k]))


def _fgcr(apply, precond, b, m, tol):
    """FGCR with restarts of m, classical Gram-Schmidt repeated once where a new vector lost more than half its norm."""
    x, r, steps, repeats = np.zeros_like(b), b.copy(), 0, 0
    while np.linalg.norm(r) > tol * np.linalg.norm(b):
        Z, W = [], []
        for k in range(m):
            z = precond(r)
            w = apply(z)
            for again in range(2):
                n0 = np.vdot(w, w).real
                cs = [np.vdot(q, w) for q, _ in W]
                for c, (q, zq) in zip(cs, W):
                    w = w - c * q
                    z = z - c * zq
                if np.vdot(w, w).real > 0.25 * n0 or not W:
                    break
                repeats += again == 0
            nw = np.linalg.norm(w)
            W.append((w / nw, z / nw))
            c = np.vdot(W[-1][0], r)
            r = r - c * W[-1][0]
            x = x + c * W[-1][1]
            steps += 1
            if np.linalg.norm(r) <= tol * np.linalg.norm(b):
                break
        r = b - apply(x)
    return x, steps, repeats


def test_repeated_pass(oracle):
    # four additive cycles near the singular point: the preconditioned vectors crowd into few directions, and later
    # ones lose most of their norm (16 of 61 steps with this source)
    case = Case("4^4/2^4", (4, 4, 4, 4), (2, 2, 2, 2), 0.16, 1.0, 0.3, 603)
    ctx = case.context()
    ctx.set_schwarz("additive")
    ctx.set_sap(4, 2, "f64")
    ctx.set_solver(16, 1e-9, 40)
    b = case.source(31)
    x, info, st = ctx.solve(dev(b))
    _, steps, repeats = _fgcr(lambda v: host(ctx.apply_D(dev(v))), lambda v: host(ctx.sap(dev(v))), b, 16, 1e-9)
    assert repeats > 0
    # the same recursion, rounded differently: the step that meets the tolerance may shift a little
    assert st == 0 and abs(info[0]["iters"] - steps) <= 0.1 * steps
    assert rel(oracle.apply_A(case.L, BC, case.U, case.C, host(x)), b) <= 1.001e-9


def test_bicgstab_steps():
    ctx = CASE.context()
    b = CASE.source(32)
    A = lambda v: host(ctx.apply_D(dev(v)))
    x, r = np.zeros_like(b), b.copy()
    r0, p, v = r.copy(), np.zeros_like(b), np.zeros_like(b)
    rho_old = alpha = omega = 1.0
    for it in range(1, 5):
        rho = np.vdot(r0, r)
        beta = (rho / rho_old) * (alpha / omega)
        p = r + beta * (p - omega * v)
        v = A(p)
        alpha = rho / np.vdot(r0, v)
        s = r - alpha * v
        t = A(s)
        omega = np.vdot(t, s) / np.vdot(t, t).real
        x = x + alpha * p + omega * s
        r = s - omega * t
        rho_old = rho
        got, info, st = ctx.solve_bicgstab(dev(b), max_iter=it, check=False)
        assert st != 0 and info["iters"] == it
        # a few hundred roundings of 1.1e-16, amplified by the condition of the recursion's scalars (< 100)
        assert rel(host(got), x) <= 1e-11
        assert abs(info["rel_residual"] - np.linalg.norm(r) / np.linalg.norm(b)) <= 1e-11
