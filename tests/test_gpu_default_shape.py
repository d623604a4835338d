"""The default pass shape at sides around the lines its rule draws (sites per
lane, pass mode, z-chunk), with both storages and stencil kinds, against the
general shape: one site per lane, mode 1, short z-chunks.  A shape changes
only the order of the lattice sums, which feed back through a: a few 1e-16 per
step of the scale factor, so fields agree to 1e-12 of their largest value; FP32
remainders then round to the same or a neighbouring value (6e-8 of the
remainder's largest, which is at most the field's)."""
import numpy as np
import pytest

import paper_1201_5029_amd as sl
import synth
from gpu_util import max_rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,model,precision,stencil", [
    (38, "preheat", "f64", None), (40, "preheat", "f64", None), (54, "preheat", "f64", None),
    (64, "preheat", "f64", None), (120, "preheat", "f64", None), (99, "preheat", "f64", None),
    (32, "oscillon", "f32", None), (52, "oscillon", "f32", None), (56, "oscillon", "f32", None),
    (88, "preheat", "f32", None), (48, "oscillon", "f64", None),
    (64, "preheat", "f64", "27"), (110, "preheat", "f32", "27"), (112, "preheat", "f32", "27"),
    (48, "oscillon", "f64", "27")])
def test_default_shape_equals_general(n, model, precision, stencil):
    r = getattr(synth, model)(n=n, precision=precision)
    r.update(fluct="white", amplitude=1e-3, seed=77, stencil=stencil)
    if model == "preheat":
        r["dt"] = 1e-4
    a, b = sl.from_recipe(r), sl.from_recipe(r)
    b.set_tile(16, 1, 3, 1)
    say("n", n, model, precision, stencil, "default", a.tile(), "general", b.tile())
    for lat in (a, b):
        lat.evolve(35, r["dt"], 4)      # a replayed graph of 32 steps and a tail
    tol = 1e-12 if precision == "f64" else 1e-6
    for got, want in zip(a.get_fields(), b.get_fields()):
        assert max_rel(got, want) < tol
    assert a.background()[1] == pytest.approx(b.background()[1], rel=1e-13 if precision == "f64" else 1e-9)
    a.close()
    b.close()
