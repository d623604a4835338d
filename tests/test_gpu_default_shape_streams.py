"""The default pass shape on both sides of the line between states that stay in
the last-level cache and states that stream, with each storage and field count,
and on the smallest sides: the sites per lane and pass mode that the rule
says, and a short run against the general shape (one site per lane, mode 1,
short chunks).  Tolerances as for the cached sides: a shape changes only the
order of the lattice sums, a few 1e-16 per step of the scale factor; FP32
remainders then round to the same or a neighbouring value."""
import pytest

import paper_1201_5029_amd as sl
import synth
from gpu_util import max_rel, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _forget_tuned_shapes():
    sl.symlat.autotune_forget()
    yield


def _recipe(model, n, precision, stencil):
    if model == "free3":
        r = dict(n=n, L=32.0, nfields=3, potential="free", params=(0.5, 0.75, 1.0), mpl=5.0,
                 phi0=(1.0, 0.9, 0.8), pi0=(0.0, 0.05, 0.1), precision=precision, dt=1e-3)
    else:
        r = getattr(synth, model)(n=n, precision=precision)
        r["dt"] = min(r["dt"], 1e-4 if model == "preheat" else 1e-3)
    r.update(fluct="white", amplitude=1e-3, seed=78, stencil=stencil)
    return r


@pytest.mark.parametrize("n,model,precision,stencil,lane", [
    # below and above 270 MB of state
    (160, "preheat", "f64", None, (2, 1)), (164, "preheat", "f64", None, (2, 7)),
    (165, "preheat", "f64", None, (1, 2)), (166, "preheat", "f64", None, (2, 7)),
    (200, "preheat", "f32", None, (2, 2)), (204, "preheat", "f32", None, (4, 2)),
    (206, "preheat", "f32", None, (2, 2)), (224, "preheat", "f32", None, (4, 6)),
    (224, "qball", "f32", None, (4, 6)), (96, "qball", "f64", None, (2, 1)),
    (200, "oscillon", "f64", None, (2, 2)), (208, "oscillon", "f64", None, (2, 7)),
    (256, "oscillon", "f32", None, (4, 2)), (288, "oscillon", "f32", None, (4, 6)),
    (160, "preheat", "f64", "27", (1, 1)), (164, "preheat", "f64", "27", (2, 1)),
    # non-temporal 27-point stores of two fields: n a multiple of 32
    (208, "preheat", "f64", "27", (2, 1)), (224, "preheat", "f64", "27", (2, 5)),
    (208, "oscillon", "f64", "27", (2, 5)), (232, "preheat", "f32", "27", (2, 1)),
    (224, "preheat", "f32", "27", (2, 5)), (205, "preheat", "f32", "27", (1, 1)),
    (64, "free3", "f64", None, (1, 1)), (144, "free3", "f64", None, (1, 1)),
    (182, "free3", "f32", "27", (1, 1)),
    # smallest sides
    (6, "preheat", "f64", None, (1, 2)), (20, "qball", "f32", None, (1, 2)),
    (24, "oscillon", "f64", "27", (1, 1)), (31, "preheat", "f32", None, (1, 2))])
def test_default_shape_equals_general(n, model, precision, stencil, lane):
    r = _recipe(model, n, precision, stencil)
    a, b = sl.from_recipe(r), sl.from_recipe(r)
    tx, vx, ty, tz, pf = a.tile()
    assert (vx, pf) == lane
    b.set_tile(16, 1, min(3, n), 1)
    say("n", n, model, precision, stencil, "default", a.tile(), "general", b.tile())
    for lat in (a, b):
        lat.evolve(3, r["dt"], 4)
    tol = 1e-12 if precision == "f64" else 1e-6
    for got, want in zip(a.get_fields(), b.get_fields()):
        assert max_rel(got, want) < tol
    assert a.background()[1] == pytest.approx(b.background()[1], rel=1e-13 if precision == "f64" else 1e-9)
    a.close()
    b.close()


@pytest.mark.parametrize("n,nf,precision", [
    (176, 4, "f64"), (176, 8, "f32"), (144, 6, "f32"), (170, 3, "f64"), (174, 5, "f32"), (200, 3, "f64"),
    (304, 5, "f32")])
def test_widths_of_several_streaming_fields(n, nf, precision):
    """More than two fields that stream through the 7-point pass: tiles of whole 16
    lanes or exact parts of a row (ragged ones, as two fields have them, took up to
    47 % longer than 64 lanes)."""
    lat = sl.Lattice(n, nf, 32.0, precision=precision)
    lat.set_potential("free", (1.0,) * nf)
    say("n", n, nf, precision, lat.tile())
    assert lat.tile()[0] % 16 == 0 or n % lat.tile()[0] == 0
    lat.close()
