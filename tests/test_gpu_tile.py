"""The tile block solve at the edges of its tiles: one to four right-hand sides (tiles of two, so a lone one, full
tiles and a remainder), both Schwarz variants (one boundary buffer, or two that alternate) and one to three cycles
(first, last and middle visits), against the oracle; and the FP32 input and output of the mixed outer solver."""
import numpy as np
import pytest

from tests.gpu_cases import BC, SAP_TOL, SITE_FACTOR, SMALL, WIDE, dev, host, rel, site_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("case", [SMALL[2], WIDE[1]], ids=repr)
@pytest.mark.parametrize("prec", ["f16", "bf16"])
@pytest.mark.parametrize("kind", ["multiplicative", "additive"])
@pytest.mark.parametrize("cycles,nrhs", [(1, 1), (2, 2), (3, 3), (2, 4)])
def test_tile_edges(case, prec, kind, cycles, nrhs, oracle):
    etas = np.stack([case.source(300 + k) for k in range(nrhs)])
    sap = oracle.sap if kind == "multiplicative" else oracle.sap_additive
    ctx = case.context()
    ctx.set_sap(cycles, 2, prec, "tile")
    ctx.set_schwarz(kind)
    got = host(ctx.sap(dev(etas)))
    for k in range(nrhs):
        want = sap(case.L, case.b, BC, case.U, case.C, case.Ci, cycles, 2, etas[k])
        err, site = site_err(got[k], want)
        assert err <= SAP_TOL[prec] and site <= SITE_FACTOR * SAP_TOL[prec], (k, err, site)


def test_tile_mixed_outer(oracle):
    case = SMALL[2]
    f = case.source(310)
    ctx = case.context()
    ctx.set_sap(case.n_cycles, case.n_mr, "f16", "tile")
    ctx.set_outer("fgcr_mixed", 0)
    x, info, st = ctx.solve(dev(f))
    assert st == 0 and rel(oracle.apply_A(case.L, BC, case.U, case.C, host(x)), f) <= 1e-10
