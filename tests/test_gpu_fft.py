"""The half-spectrum transforms against numpy's, through the spectra they
feed: sides of every plan class (powers of two; factors 3 and 5; 7, larger
primes and sides of a single stage), odd and ragged, both storage precisions,
one to three fields (interleaved and separate arrays, and the scratch pieces
each leaves), and the sides above 256 that run with 512 threads."""
import math

import numpy as np
import pytest

import oracle
import paper_1201_5029_amd as sl
import synth
from gpu_util import gpu_lattice, oracle_lattice, say

pytestmark = pytest.mark.gpu


def _check(n, nf, precision, seed, stencil=None):
    m2 = tuple(0.5 + 0.3 * i for i in range(nf))
    base, pib = [0.7 - 0.2 * i for i in range(nf)], [0.1 * i for i in range(nf)]
    phi, pi = synth.gaussian_state(n, nf, seed, phi_base=base, phi_amp=1e-2, pi_base=pib, pi_amp=1e-2)
    g = gpu_lattice(n, 8.0, "free", m2, phi, pi, precision=precision, mpl=2.0, stencil=stencil)
    g.evolve(1, 0.01 * min(1.0, 32.0 / n), 2)         # leaves a drift pending
    phi, pi = g.get_fields()
    o = oracle_lattice(n, 8.0, "free", m2, phi, pi, mpl=2.0, stencil=stencil)
    _, a, _ = g.background()
    o.a = a
    nb = int(math.ceil(math.sqrt(3) * n / 2)) + 2
    field = nf - 1
    k, pf, pe, pn, cnt, m2g = g.spectra(field, nb)
    k1, p1, c1 = g.spectrum(field, nb)
    after = g.get_fields()
    assert np.array_equal(after[0], phi) and np.array_equal(after[1], pi)  # the state is untouched
    ko, pfo, peo, pno, co, m2o = oracle.mode_spectra(o, field, nb)
    say("n", n, "nf", nf, precision, "pf[1:4]", pf[1:4], pfo[1:4])
    assert np.array_equal(cnt, co) and np.array_equal(c1, co)
    assert m2g == pytest.approx(m2o, rel=1e-12)
    for got, ref in ((k, ko), (k1, ko)):
        np.testing.assert_allclose(got, ref, rtol=1e-12)
    for got, ref in ((pf, pfo), (pe, peo), (pn, pno), (p1, pfo)):
        np.testing.assert_allclose(got, ref, rtol=1e-9, atol=1e-12 * np.abs(ref).max())
    g.evolve(1, 0.01 * min(1.0, 32.0 / n), 2)         # the next pass overwrites the scratch
    assert np.isfinite(g.energies()["rho"])
    g.close()


@pytest.mark.parametrize("n", [4, 5, 6, 7, 8, 9, 11, 13, 14, 22, 25, 27, 31, 32, 33, 36, 42, 49, 50, 64,
                               75, 77, 96, 97, 100, 121, 128])
def test_spectra_of_every_plan_class(n):
    nf, precision = 1 + n % 3, ("f32", "f64")[n % 2]
    _check(n, nf, precision, 700 + n, oracle.STENCIL_27 if n % 4 == 1 else None)


@pytest.mark.parametrize("n,precision", [(32, "f32"), (33, "f64"), (270, "f32"), (264, "f64"), (320, "f32")])
def test_spectra_one_field(n, precision):
    """One field: FP32 arrays are shorter than the half spectrum (it goes on
    in the partial-sum buffer, or at 320 in an allocation)."""
    _check(n, 1, precision, 800 + n)


@pytest.mark.parametrize("n", [512, 1024])
def test_largest_sides_parseval(n):
    """Sum of the bins = lattice variance (512 threads, LDS above 64 KB)."""
    lat = sl.Lattice(n, 1, 64.0, precision="f32")
    lat.set_potential("free", (1.0,))
    lat.init_fluctuations((0.5,), (0.0,), "white", 1e-3, 11)
    _, p, c = lat.spectrum(0, 2048)
    var = lat.energies()["var"][0]
    say("n", n, "sum", float((p * c).sum()), "var", var)
    assert int(c.sum()) == n ** 3 - 1
    assert float((p * c).sum()) == pytest.approx(var, rel=1e-9)
    lat.close()
