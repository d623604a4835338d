"""Host arrays through the ring of pinned slots: a linearized handle's fields in
and straight out again at sizes below, at and above the size where the ring
takes over (8 MiB both arrays together), with a last chunk of any length, twice
with different arrays (slots reused).  What comes back went through a forward
and an inverse transform, whose rounding is a few 1e-16 of the largest value
per level (at most 20 levels): 1e-13 of it holds."""
import numpy as np
import pytest

import paper_1201_5029_amd as sl
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nf", [(16, 1), (63, 2), (64, 2), (65, 2), (81, 1), (100, 3)])
def test_fields_in_and_out(n, nf):
    lin = sl.Linear(n, nf, 0.5 * n)
    lin.set_potential("free", [1.0 + i for i in range(nf)])
    rng = np.random.default_rng(4400 + n)
    for rep in range(2):
        phi = rng.standard_normal((nf, n, n, n))
        pi = 3.0 + rng.standard_normal((nf, n, n, n))
        lin.set_fields(phi, pi)
        got = lin.get_fields()
        for g, want in zip(got, (phi, pi)):
            err = np.abs(g - want).max() / np.abs(want).max()
            say("n", n, "fields", nf, "pass", rep, "err", err)
            assert err < 1e-13
    lin.close()
