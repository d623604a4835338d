"""The observables' forward-bond walk where its tiles change form: one or two
sites per lane (odd or even n, storage), rows just short of, at and just over
one tile and one wavefront, z-chunks of one plane, with the state as set.
The oracle sums all six neighbours.  Tolerance: fields of order 1 with
differences of order 1e-2 carry a rounding error of about 1e-14 of a bond, the
sums over at most 130 planes in a row and the divided totals less than that
times 130: 1e-10 holds both with a margin."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import gpu_lattice, oracle_lattice, say

pytestmark = pytest.mark.gpu

MODELS = {
    "chaotic2": ((1.0, 9312.25), (1.0, 0.5), 1.0335292),
    "qball": ((1.0, -0.1, 1.0), (1.0, 0.5), 1.0),
    "oscillon": ((1.0, 1.0, 0.2), (0.8,), 335.41),
}

# weights of eq. (2.7): the isotropic 27-point member and one with unrelated values
STENCILS = {"iso": oracle.STENCIL_27, "wide": (-(6 * 0.4 + 12 * 0.1 + 8 * 0.05), 0.4, 0.1, 0.05)}


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


@pytest.mark.parametrize("n,kind,precision,stencil", [
    (4, "chaotic2", "f64", "iso"), (5, "oscillon", "f64", "iso"), (63, "qball", "f64", "iso"),
    (64, "chaotic2", "f64", "iso"), (66, "oscillon", "f64", "wide"), (129, "chaotic2", "f64", "iso"),
    (65, "qball", "f32", "wide"), (96, "chaotic2", "f32", "iso")])
def test_bond_sums_27(n, kind, precision, stencil):
    """The 13 forward bonds of the general stencil (the oracle sums all 26
    neighbours): a weight of each class, tiles with ragged edges, and a member of
    the family with its own weights."""
    params, base, mpl = MODELS[kind]
    nf = len(base)
    c = STENCILS[stencil]
    phi, pi = synth.gaussian_state(n, nf, 9300 + n, phi_base=list(base), phi_amp=1e-2, pi_amp=1e-2)
    g = gpu_lattice(n, 0.5 * n, kind, params, phi, pi, precision=precision, mpl=mpl, stencil=c)
    if precision == "f32":      # the oracle sees the values the library stores
        phi, pi = g.get_fields()
    o = oracle_lattice(n, 0.5 * n, kind, params, phi, pi, mpl=mpl, stencil=c)
    eg, eo = g.energies(), o.energies()
    say("n", n, kind, precision, stencil, "rho", eg["rho"], eo["rho"], "grad", eg["grad"][:nf],
        eo["grad"][:nf])
    assert g.background()[2] == pytest.approx(o.p_a, rel=1e-10)
    for k in ("rho", "pot", "p_a", "h_total"):
        assert eg[k] == pytest.approx(eo[k], rel=1e-10, abs=1e-10 * abs(eo["rho"]) * n ** 3), k
    for k in ("kin", "grad", "mean", "var"):
        np.testing.assert_allclose(eg[k][:nf], eo[k][:nf], rtol=1e-10, err_msg=k)
    g.close()
