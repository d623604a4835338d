"""sl_spectra on sides whose binning pass takes more than 64 KB of LDS, up to the
largest (134 KB), by Parseval: free fields that fluctuate around zero, on a
static background, whose mode energies add up to the density and whose powers to
the variance.  Sums over 1e9 modes in FP64, most of them plain over at most 1e6
terms: 1e-9."""
import pytest

import paper_1201_5029_amd as sl
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nf,precision,stencil", [
    (360, 1, "f64", "27"), (512, 1, "f64", "7"), (512, 2, "f32", "27"), (1024, 1, "f32", "7")])
def test_mode_energies_add_up(n, nf, precision, stencil):
    m2 = (1.0, 2.0)[:nf]
    lat = sl.Lattice(n, nf, n / 16.0, precision=precision, expand=False)
    lat.set_potential("free", m2)
    lat.set_stencil(stencil)
    lat.init_fluctuations((0.0,) * nf, (0.0,) * nf, "white", 1e-3, 19)
    lat.evolve(2, 0.005, 2)           # the momenta fluctuate, a drift is pending
    e = lat.energies()
    for i in range(nf):
        k, pf, pe, pn, count, m2eff = lat.spectra(i, 2048)
        var = float((pf * count).sum())
        rho = float((pe * count).sum())
        want = e["kin"][i] + e["grad"][i] + 0.5 * m2[i] * (e["var"][i] + e["mean"][i] ** 2)
        say("n", n, "field", i, "var", var, e["var"][i], "rho", rho, want, "kin", e["kin"][i])
        assert int(count.sum()) == n ** 3 - 1 and m2eff == pytest.approx(m2[i], rel=1e-14)
        assert e["kin"][i] > 1e-3 * rho
        assert var == pytest.approx(e["var"][i], rel=1e-9)
        assert rho == pytest.approx(want, rel=1e-9)
    lat.close()
