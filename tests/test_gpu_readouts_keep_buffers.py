"""Read-outs of a lattice on the caller's arrays leave all four of them as they
are, the pair that does not hold the state included (it keeps the stage before),
and give what a lattice that owns its arrays gives: the bin sums of the spectra
use LDS atomics, whose order varies in the last bits."""
import ctypes

import numpy as np
import pytest

import paper_1201_5029_amd as sl
import synth
from gpu_util import say

pytestmark = pytest.mark.gpu


def _hip():
    sl.load()                                   # the library's own runtime is loaded
    hip = ctypes.CDLL("libamdhip64.so.7")
    hip.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
    hip.hipFree.argtypes = [ctypes.c_void_p]
    hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    return hip


@pytest.mark.parametrize("n,precision", [(16, "f64"), (33, "f32"), (48, "f64"), (96, "f32")])
def test_readouts_leave_the_callers_arrays(n, precision):
    hip = _hip()
    r = synth.preheat(n=n, precision=precision, seed=41)
    nf, elem = r["nfields"], 8 if precision == "f64" else 4
    nbytes = nf * n ** 3 * elem
    bufs = []
    for _ in range(4):
        p = ctypes.c_void_p()
        assert hip.hipMalloc(ctypes.byref(p), nbytes) == 0
        bufs.append(p.value)

    def arrays():
        host = [np.empty(nf * n ** 3 * elem, dtype=np.uint8) for _ in bufs]
        for h, b in zip(host, bufs):
            assert hip.hipMemcpy(h.ctypes.data, b, nbytes, 2) == 0
        return host
    try:
        own = sl.Lattice(n, nf, r["L"], precision=precision, mpl=r["mpl"])
        ext = sl.Lattice(n, nf, r["L"], precision=precision, mpl=r["mpl"], buffers=bufs)
        for lat in (own, ext):
            lat.set_potential(r["potential"], r["params"])
            lat.init_fluctuations(r["phi0"], r["pi0"], "vacuum", 1e-3, 41)
            lat.evolve(3, 1e-3, 4)
            lat.synchronize()
        before = arrays()
        got = [ext.spectra(1, n), ext.spectrum(0, n)]
        ext.energies()
        ext.get_fields()
        after = arrays()
        say("n", n, precision, "changed bytes", [int((x != y).sum()) for x, y in zip(before, after)])
        for x, y in zip(before, after):
            assert np.array_equal(x, y)
        for a, b in zip(got, [own.spectra(1, n), own.spectrum(0, n)]):
            for x, y in zip(a, b):
                np.testing.assert_allclose(x, y, rtol=1e-9, atol=1e-12 * np.max(np.abs(y)))
        ext.close()
        own.close()
    finally:
        for b in bufs:
            hip.hipFree(b)
