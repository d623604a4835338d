"""Vacuum states in units whose side cubed is no double: with no mass term f_n
goes as A/L, so that side and amplitude scaled by one power of two give the same
fields; every factor of the scaled modes is exact but for one ulp of the
variance, whose root enters: 1e-15 of the largest value."""
import numpy as np
import pytest

import paper_1201_5029_amd as sl
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("power", [-360, -100, 100, 360])
@pytest.mark.parametrize("n", [8, 15])
def test_vacuum_state_scales_with_the_side(n, power):
    def draw(scale):
        lat = sl.Lattice(n, 1, 8.0 * scale, expand=False)
        lat.set_potential("free", (0.0,))
        lat.init_fluctuations((0.5,), (0.25,), "vacuum", 1e-3 * scale, 77)
        phi, pi = lat.get_fields()
        lat.close()
        return phi, pi
    (want, _), (phi, pi) = draw(1.0), draw(2.0 ** power)
    peak = np.abs(want - 0.5).max()
    say("n", n, "power", power, "peak", peak, "difference", np.abs(phi - want).max())
    assert peak > 1e-5 and np.abs(phi - want).max() <= 1e-15 * 0.51
    assert np.all(pi == 0.25)
