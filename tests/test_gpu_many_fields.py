"""Observables with the most fields: the general-stencil walk keeps three planes
of every field in LDS, with seven and eight fields more than 64 KB (such a
kernel has to be told).  Against the oracle; tolerance as for fewer fields
(1e-10: differences of 1e-2 on fields of order 1, at most 65 planes in a row)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import gpu_lattice, oracle_lattice, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nf,precision,stencil", [
    (6, 7, "f64", "27"), (65, 7, "f64", "27"), (20, 8, "f32", "27"), (66, 8, "f64", "27"), (33, 8, "f64", "7"),
    (64, 7, "f32", "7")])
def test_observables_of_many_fields(n, nf, precision, stencil):
    m2 = tuple(0.5 + 0.25 * i for i in range(nf))
    base = [1.0 - 0.2 * i for i in range(nf)]
    c = oracle.STENCIL_27 if stencil == "27" else oracle.STENCIL_7
    phi, pi = synth.gaussian_state(n, nf, 9500 + n, phi_base=base, phi_amp=1e-2, pi_amp=1e-2)
    g = gpu_lattice(n, 0.5 * n, "free", m2, phi, pi, precision=precision, stencil=c)
    if precision == "f32":      # the oracle sees the values the library stores
        phi, pi = g.get_fields()
    o = oracle_lattice(n, 0.5 * n, "free", m2, phi, pi, stencil=c)
    eg, eo = g.energies(), o.energies()
    say("n", n, nf, precision, stencil, "rho", eg["rho"], eo["rho"])
    assert g.background()[2] == pytest.approx(o.p_a, rel=1e-10)
    for k in ("rho", "pot", "p_a"):
        assert eg[k] == pytest.approx(eo[k], rel=1e-10), k
    for k in ("kin", "grad", "mean", "var"):
        np.testing.assert_allclose(eg[k][:nf], eo[k][:nf], rtol=1e-10, err_msg=k)
    g.close()
