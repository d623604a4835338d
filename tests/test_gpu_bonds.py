"""The observables' forward-bond walk where its tiles change form: one or two
sites per lane (odd or even n, storage), rows just short of, at and just over
one tile and one wavefront, z-chunks of one plane, with the state as set.
The oracle sums all six neighbours.  Tolerance: fields of order 1 with
differences of order 1e-2 carry a rounding error of about 1e-14 of a bond, the
sums over at most 130 planes in a row and the divided totals less than that
times 130: 1e-10 holds both with a margin."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_lattice, oracle_lattice, say

pytestmark = pytest.mark.gpu

MODELS = {
    "chaotic2": ((1.0, 9312.25), (1.0, 0.5), 1.0335292),
    "qball": ((1.0, -0.1, 1.0), (1.0, 0.5), 1.0),
    "oscillon": ((1.0, 1.0, 0.2), (0.8,), 335.41),
}


@pytest.mark.parametrize("n,kind,precision", [
    (4, "qball", "f64"), (6, "chaotic2", "f64"), (63, "qball", "f64"), (64, "oscillon", "f64"),
    (126, "qball", "f64"), (128, "oscillon", "f64"), (129, "chaotic2", "f64"),
    (64, "qball", "f32"), (65, "oscillon", "f32"), (128, "chaotic2", "f32")])
def test_bond_sums(n, kind, precision):
    params, base, mpl = MODELS[kind]
    nf = len(base)
    phi, pi = synth.gaussian_state(n, nf, 9100 + n, phi_base=list(base), phi_amp=1e-2, pi_amp=1e-2)
    g = gpu_lattice(n, 0.5 * n, kind, params, phi, pi, precision=precision, mpl=mpl)
    if precision == "f32":      # the oracle sees the values the library stores
        phi, pi = g.get_fields()
    o = oracle_lattice(n, 0.5 * n, kind, params, phi, pi, mpl=mpl)
    eg, eo = g.energies(), o.energies()
    say("n", n, kind, precision, "rho", eg["rho"], eo["rho"], "grad", eg["grad"][:nf],
        eo["grad"][:nf])
    assert g.background()[2] == pytest.approx(o.p_a, rel=1e-10)
    for k in ("rho", "pot", "p_a"):
        assert eg[k] == pytest.approx(eo[k], rel=1e-10), k
    for k in ("kin", "grad", "mean", "var"):
        np.testing.assert_allclose(eg[k][:nf], eo[k][:nf], rtol=1e-10, err_msg=k)
    g.close()
