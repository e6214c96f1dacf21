"""Launches of many systems of a small lattice with 4^4 domains, which take another block-solve kernel than one system
does (more than 256 workgroups): the bits of each system alone, in every precision, first, middle and last visits, both
Schwarz variants, with right-hand sides of one lattice and with lattices of a batch."""
import numpy as np
import pytest

from tests.gpu_cases import Case, dev, host

pytestmark = pytest.mark.gpu

CASE = Case("8^4/4^4", (8, 8, 8, 8), (4, 4, 4, 4), 0.1365, 1.7, 0.6, 701)   # 8 workgroups a colour
ODD = Case("16x8x8x24/4^4", (16, 8, 8, 24), (4, 4, 4, 4), 0.13, 1.5, 0.5, 702)   # 48
NRHS = 33


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.fixture(scope="module")
def sources():
    return dev(np.stack([CASE.source(800 + k) for k in range(NRHS)]))


@pytest.mark.parametrize("kind", ["multiplicative", "additive"])
@pytest.mark.parametrize("prec", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("cycles,mr", [(1, 1), (3, 3)])
def test_sap_of_many_right_hand_sides(kind, prec, cycles, mr, sources):
    ctx = CASE.context()
    ctx.set_schwarz(kind)
    ctx.set_sap(cycles, mr, prec)
    got = host(ctx.sap(sources))
    for k in (0, 1, 16, NRHS - 1):
        assert np.array_equal(host(ctx.sap(sources[k].contiguous())), got[k]), k


@pytest.mark.parametrize("outer", ["fgcr", "fgcr_mixed"])
def test_solve_of_a_batch(outer):
    # 8 systems of 48 workgroups: 384; as they converge the launches fall below 257
    from paper_1412_2629_amd import ddqcd
    ctxs = []
    for _ in range(2):
        c = ODD.context()
        c.set_sap(4, 4, "f16")
        c.set_outer(outer)
        ctxs.append(c)
    bs = [dev(ODD.source(850 + k)) for k in range(8)]
    xs, infos, st = ddqcd.solve_batch([ctxs[k % 2] for k in range(8)], bs)
    assert st == 0
    for k in (0, 3, 7):
        x, info, s = ctxs[0].solve(bs[k])
        assert s == 0 and info[0]["iters"] == infos[k]["iters"] and np.array_equal(host(x), host(xs[k])), k
