"""The block solve with two threads per site, on both sides of the lattice size at which it gives way to the one with
one thread per site (256 workgroups a colour), for each domain shape that has it, in one, two and three cycles (first,
last and middle visits), both Schwarz variants, against the oracle."""
import numpy as np
import pytest

from tests.gpu_cases import BC, SAP_TOL, SITE_FACTOR, Case, dev, host, rel, site_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


EDGE = [   # the largest lattice of two threads per site, the smallest of one
    Case("16x16x16x32/4^4", (16, 16, 16, 32), (4, 4, 4, 4), 0.13, 1.5, 0.5, 401),
    Case("16x16x16x40/4^4", (16, 16, 16, 40), (4, 4, 4, 4), 0.13, 1.5, 0.5, 402),
    Case("16x16x16x16/2^4", (16, 16, 16, 16), (2, 2, 2, 2), 0.13, 1.5, 0.5, 403),
    Case("16x16x16x20/2^4", (16, 16, 16, 20), (2, 2, 2, 2), 0.13, 1.5, 0.5, 404),
    Case("24x24x8x32/6x6x2x4", (24, 24, 8, 32), (6, 6, 2, 4), 0.13, 1.5, 0.5, 405),
    Case("24x24x8x40/6x6x2x4", (24, 24, 8, 40), (6, 6, 2, 4), 0.13, 1.5, 0.5, 406),
]


@pytest.mark.parametrize("case", EDGE, ids=repr)
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
def test_edge_of_rule(case, prec, oracle):
    if prec == "f64" and case.b != (2, 2, 2, 2):
        pytest.skip("FP64 has two threads per site on 2^4 domains only")
    eta = case.source(7)
    want = oracle.sap(case.L, case.b, BC, case.U, case.C, case.Ci, 2, 2, eta)
    ctx = case.context()
    ctx.set_sap(2, 2, prec)
    err, site = site_err(host(ctx.sap(dev(eta))), want)
    assert err <= SAP_TOL[prec] and site <= SITE_FACTOR * SAP_TOL[prec], (err, site)


SMALL_SPLIT = [
    Case("4x8x4x4/2^4", (4, 8, 4, 4), (2, 2, 2, 2), 0.13, 1.5, 0.5, 411),
    Case("8x16x8x8/4^4", (8, 16, 8, 8), (4, 4, 4, 4), 0.13, 1.5, 0.5, 412),
    Case("12x24x4x8/6x6x2x4", (12, 24, 4, 8), (6, 6, 2, 4), 0.13, 1.5, 0.5, 413),
]


@pytest.mark.parametrize("case", SMALL_SPLIT, ids=repr)
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("kind", ["multiplicative", "additive"])
def test_visits(case, prec, kind, oracle):
    if prec == "f64" and case.b != (2, 2, 2, 2):
        pytest.skip("FP64 has two threads per site on 2^4 domains only")
    eta = case.source(8)
    sap = oracle.sap if kind == "multiplicative" else oracle.sap_additive
    ctx = case.context()
    ctx.set_schwarz(kind)
    for cycles in (1, 3):
        want = sap(case.L, case.b, BC, case.U, case.C, case.Ci, cycles, 3, eta)
        ctx.set_sap(cycles, 3, prec)
        got = host(ctx.sap(dev(eta)))
        err, site = site_err(got, want)
        assert err <= SAP_TOL[prec] and site <= SITE_FACTOR * SAP_TOL[prec], (cycles, err, site)
        assert np.array_equal(host(ctx.sap_noalloc(dev(eta))), got)


def test_split_mixed_outer(oracle):
    case = SMALL_SPLIT[1]
    f = case.source(9)
    ctx = case.context("f16")
    ctx.set_outer("fgcr_mixed", 0)
    x, info, st = ctx.solve(dev(f))
    assert st == 0 and rel(oracle.apply_A(case.L, BC, case.U, case.C, host(x)), f) <= 1e-10
