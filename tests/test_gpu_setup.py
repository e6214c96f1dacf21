"""The inverse of the odd sites' clover blocks where its elimination exchanges rows (a clover coefficient far above the
physical range: the diagonal no longer dominates) and where it does not, seen through one block solve in FP64."""
import numpy as np
import pytest

from tests.gpu_cases import BC, SITE_FACTOR, Case, dev, host, site_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _blocks(C):
    C = np.asarray(C)
    return np.concatenate([C[:, :6, :6], C[:, 6:, 6:]])


def _exchanges(M):
    n = 0
    for a in M.copy():
        for c in range(6):
            p = c + int(np.argmax(np.abs(a[c:, c])))
            if p != c:
                n += 1
                a[[c, p]] = a[[p, c]]
            a[c] /= a[c, c]
            for r in range(6):
                if r != c:
                    a[r] -= a[r, c] * a[c]
    return n


@pytest.mark.parametrize("L,b", [((4, 4, 4, 4), (2, 2, 2, 2)), ((8, 8, 8, 8), (4, 4, 4, 4))])
@pytest.mark.parametrize("csw", [1.5, 20.0])
def test_clover_inverse(L, b, csw, oracle):
    case = Case(f"{L}/{b}", L, b, 0.13, csw, 0.5, 701)
    M = _blocks(case.C)
    assert (_exchanges(M[:256]) > 0) == (csw > 2)
    # an elimination of six rows, some tens of roundings of 1.1e-16 each amplified by the worst block's condition
    # (1.9 and some thousands), applied twice in a block solve of one step
    tol = 100 * 2.0 ** -53 * np.linalg.cond(M).max()
    eta = case.source(5)
    want = oracle.sap(case.L, case.b, BC, case.U, case.C, case.Ci, 1, 1, eta)
    ctx = case.context()
    ctx.set_sap(1, 1, "f64")
    err, site = site_err(host(ctx.sap(dev(eta))), want)
    assert err <= tol and site <= SITE_FACTOR * tol, (err, site, tol)
