"""Rounding of the observables' sums over long chunks, with a general stencil: a
homogeneous state, whose lattice sums are its values, at a side where a lane
adds 128 planes.  Every lane then rounds alike, so that a plain sum's error
(1e-15 to 3e-15 of the total for these values, found on the CPU) is not averaged
away.  Tolerance: a compensated sum of equal terms leaves the rounding of the
term itself and of the divided total, a few 1.1e-16: 5e-16."""
import math
from fractions import Fraction

import pytest

import paper_1201_5029_amd as sl
from gpu_util import say

pytestmark = pytest.mark.gpu

MOMENTA = (0.9592604673872155, 0.46100610092742506, 0.36606042609212264, 0.09131292583870107)


def _plain_error(p, count):
    """Relative error of count terms p^2 added one by one with fused multiply-adds."""
    s = 0.0
    for _ in range(count):
        s = float(Fraction(p) * Fraction(p) + Fraction(s))
    return float(Fraction(s) / (count * Fraction(p) ** 2) - 1)


@pytest.mark.parametrize("p", MOMENTA)
def test_sums_of_a_long_chunk(p):
    n = 256
    lat = sl.Lattice(n, 1, 64.0, expand=False)
    lat.set_potential("free", (1.0,))
    lat.set_stencil("27")
    lat.init_fluctuations((p,), (p,), "none")
    e = lat.energies()
    want = float(Fraction(p) * Fraction(p) / 2)
    say("p", p, "plain sum's error", _plain_error(p, 128), "kin", e["kin"][0] / want - 1,
        "pot", e["pot"] / want - 1)
    assert abs(_plain_error(p, 128)) > 2.5e-15
    assert e["kin"][0] == pytest.approx(want, rel=5e-16, abs=0.0)
    assert e["pot"] == pytest.approx(want, rel=5e-16, abs=0.0)
    assert e["mean"][0] == p and e["var"][0] == 0.0 and e["grad"][0] == 0.0
    assert math.isfinite(e["rho"])
    lat.close()


@pytest.mark.parametrize("p", (0.8868600418849901, 0.4873891512036095, 0.6978830298032184))
def test_sites_of_a_lane_are_summed_apart(p):
    """The 7-point walk adds a lane's terms plainly over its chunk, 512 planes at
    this side: one site's worth, not those of both sites of a lane, whose 1024
    terms are 2e-14 to 3e-14 off for these values where 512 are less than 4e-15."""
    n = 512
    one, both = abs(_plain_error(p, n)), abs(_plain_error(p, 2 * n))
    lat = sl.Lattice(n, 1, 64.0, expand=False)
    lat.set_potential("free", (1.0,))
    lat.init_fluctuations((0.5,), (p,), "none")
    kin = lat.energies()["kin"][0]
    want = float(Fraction(p) * Fraction(p) / 2)
    say("p", p, "plain errors", one, both, "kin", kin / want - 1)
    assert both > one + 1.5e-14
    assert kin == pytest.approx(want, rel=one + 5e-16, abs=0.0)
    lat.close()
