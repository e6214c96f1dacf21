"""Which block-solve kernel serves a call (csrc/dd_form.h), compiled for the CPU."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1412_2629_amd", "csrc")
P64, P32, P16, PB16 = range(4)
LANE, TILE_VALU, MFMA_F32, MFMA_BF16, SPLIT, HALVES = range(6)

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "dd_form.h"
int main(int, char **v)
{
    const int form = dd::sap_kernel_form(atoi(v[1]), atoi(v[2]), atoi(v[3]), atol(v[4]));
    printf("%d\n", v[5] ? dd::sap_launch_form(atoi(v[1]), form, atol(v[5])) : form);
}
"""


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    d = tmp_path_factory.mktemp("form")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "main.cpp"), "-o", exe], check=True)
    return lambda *a: int(subprocess.run([exe, *map(str, a)], check=True, capture_output=True, text=True).stdout)


SIZES = [1, 256, 257, 512, 513, 100000]


@pytest.mark.parametrize("workgroups", SIZES)
def test_forms_that_hold_at_every_size(form, workgroups):
    for prec in (P32, P16, PB16):
        assert form(288, prec, LANE, workgroups) == SPLIT     # one thread per site is slower there at every size
        assert form(512, prec, LANE, workgroups) == LANE      # 512 sites have two waves per SIMD
    assert form(16, P64, LANE, workgroups) == SPLIT           # the only FP64 kernel of 16 sites
    for sites in (256, 512):
        assert form(sites, P64, LANE, workgroups) == LANE     # the only one of larger domains
    for product in (TILE_VALU, MFMA_F32, MFMA_BF16):
        assert form(256, P16, product, workgroups) == product


@pytest.mark.parametrize("prec", [P32, P16, PB16])
def test_a_full_launch_of_small_lattices_has_one_thread_per_site(form, prec):
    # lattices of 8, 128 and 256 workgroups a colour: two threads per site until the launch holds more than 256
    for lattice in (8, 128, 256):
        assert form(256, prec, LANE, lattice, lattice) == SPLIT
        assert form(256, prec, LANE, lattice, 256) == SPLIT
        for launch in (257, 264, 3072):
            assert form(256, prec, LANE, lattice, launch) == HALVES
    # a larger lattice keeps its own order of sums, other domains their kernel
    assert form(256, prec, LANE, 257, 257) == LANE
    assert form(512, prec, LANE, 8, 3072) == LANE
    assert form(288, prec, LANE, 8, 3072) == SPLIT
    assert form(16, prec, LANE, 8, 3072) == SPLIT
    assert form(256, P64, LANE, 8, 3072) == LANE
    assert form(256, P16, TILE_VALU, 8, 3072) == TILE_VALU
