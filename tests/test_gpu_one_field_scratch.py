"""Spectra and vacuum states of one FP32 field, whose two spare arrays are short
of a half spectrum: the rest goes to the partial-sum buffer, so that a call takes
no device memory.  A second thread watches the free memory while calls run; an
allocation shows as a dip of the half spectrum's 8 n^3 bytes."""
import threading

import numpy as np
import pytest

import paper_1201_5029_amd as sl
from gpu_util import say

pytestmark = pytest.mark.gpu


def _lattice(n, precision="f32"):
    lat = sl.Lattice(n, 1, 20.0, precision=precision)
    lat.set_potential("free", (1.0,))
    lat.init_fluctuations((0.5,), (0.1,), "vacuum", 1e-3, 5)
    return lat


def _least_free(calls):
    low, stop = [sl.device_memory()[0]], threading.Event()

    def watch():
        while not stop.is_set():
            low[0] = min(low[0], sl.device_memory()[0])
    t = threading.Thread(target=watch)
    t.start()
    try:
        for f in calls:
            f()
    finally:
        stop.set()
        t.join()
    return low[0]


@pytest.mark.parametrize("n", [128, 144, 160, 192, 256, 270, 300, 320, 384, 512])
def test_no_device_memory_is_taken(n):
    lat = _lattice(n)
    calls = [lambda: lat.spectrum(0, 2048), lambda: lat.spectra(0, 2048),
             lambda: lat.init_fluctuations((0.5,), (0.1,), "vacuum", 1e-3, 5)]
    for f in calls:
        f()
    free = sl.device_memory()[0]
    low = _least_free(calls * 30)
    say("n", n, "dip", free - low, "half spectrum", 8 * n ** 3)
    assert free - low < 4 * n ** 3
    lat.close()


@pytest.mark.parametrize("n", [128, 160, 256, 384])
def test_one_field_scratch_layouts(n):
    """Padded rows, unpadded ones and sides far into the partial-sum buffer, against the FP64
    lattice, which has room for padded rows everywhere: the same modes, stored
    in FP32 remainders (6e-8 of the largest)."""
    a, b = _lattice(n), _lattice(n, "f64")
    fa, fb = a.get_fields()[0], b.get_fields()[0]
    peak = np.abs(fb - 0.5).max()
    say("n", n, "peak", peak, "difference", np.abs(fa - fb).max())
    assert np.abs(fa - fb).max() <= 1e-7 * peak
    for x, y in zip(a.spectra(0, 2048), b.spectra(0, 2048)):
        np.testing.assert_allclose(x, y, rtol=1e-5, atol=1e-9 * np.max(np.abs(y)))
    pa, pb = a.spectrum(0, 2048), b.spectrum(0, 2048)
    assert np.array_equal(pa[2], pb[2])
    np.testing.assert_allclose(pa[1], pb[1], rtol=1e-5, atol=1e-9 * pb[1].max())
    a.close()
    b.close()
