"""The operator on both sides of the launch size at which whole domains per workgroup take over from one thread per
site (256 workgroups of 256 sites), with more right-hand sides than one launch holds (16), on domains without a
whole-domain kernel and on a lattice of one workgroup: against the oracle, and with the same bits for a right-hand
side whatever shares its launch."""
import numpy as np
import pytest

from tests.gpu_cases import A_TOL, BC, SITE_FACTOR, Case, dev, host, site_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


CASES = [   # 32 workgroups a right-hand side (8 and 9: the two sides of the rule), 36 and 1 in the last two
    Case("16x8x8x8/2^4", (16, 8, 8, 8), (2, 2, 2, 2), 0.13, 1.5, 0.5, 501),
    Case("16x8x8x8/4^4", (16, 8, 8, 8), (4, 4, 4, 4), 0.13, 1.5, 0.5, 502),
    Case("16x8x8x8/8x4^3", (16, 8, 8, 8), (8, 4, 4, 4), 0.13, 1.5, 0.5, 503),
    Case("8x8x8x16/4^3x8", (8, 8, 8, 16), (4, 4, 4, 8), 0.13, 1.5, 0.5, 504),
    Case("24x12x4x8/6x6x2x4", (24, 12, 4, 8), (6, 6, 2, 4), 0.13, 1.5, 0.5, 505),
    Case("4^4/2^4", (4, 4, 4, 4), (2, 2, 2, 2), 0.13, 1.5, 0.5, 506),
]


@pytest.mark.parametrize("case", CASES, ids=repr)
@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
def test_right_hand_sides_of_a_launch(case, prec, oracle):
    ctx = case.context()
    psi = np.stack([case.source(20 + k) for k in range(17)])
    all17 = host(ctx.apply_D(dev(psi), prec))
    for k in (0, 8, 16):
        err, site = site_err(all17[k], oracle.apply_A(case.L, BC, case.U, case.C, psi[k]))
        assert err <= A_TOL[prec] and site <= SITE_FACTOR * A_TOL[prec], (k, err, site)
    for n in (1, 8, 9):
        assert np.array_equal(host(ctx.apply_D(dev(psi[:n]), prec)), all17[:n]), n


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
def test_output_shifted_into_input(prec):
    case = CASES[1]
    ctx = case.context()
    psi = dev(np.stack([case.source(20 + k) for k in range(3)]))
    want = host(ctx.apply_D(psi[1:].clone(), prec))
    ctx.apply_D(psi[1:], prec, psi[:2])
    assert np.array_equal(host(psi[:2]), want)
