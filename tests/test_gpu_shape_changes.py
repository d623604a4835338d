"""The pass shape after a change of the stencil kind: it is chosen anew for the
new kernel, and a z-chunk length given by hand stays only where its tiles number
no more than the partial-sum buffer has records for."""
import math

import pytest

import paper_1201_5029_amd as sl
from gpu_util import say

pytestmark = pytest.mark.gpu

MOST_TILES = 65536


@pytest.fixture(autouse=True)
def _forget_tuned_shapes():
    sl.symlat.autotune_forget()
    yield
    sl.symlat.autotune_forget()


def _tiles(n, shape):
    tx, vx, ty, tz, _ = shape
    return math.ceil(n / (tx * vx)) * math.ceil(n / ty) * math.ceil(n / tz)


@pytest.mark.parametrize("tz", [2, 3, 16])
def test_given_chunk_within_the_tile_limit(tz):
    """512^3, two FP32 fields: four sites per lane and two planes a chunk make
    exactly 65536 tiles, the 27-point pass's two sites per lane twice as many.
    No pass is launched."""
    n = 512
    lat = sl.Lattice(n, 2, 40.0, precision="f32")
    lat.set_potential("chaotic2", (1.0, 100.0))
    lat.set_tile(64, 4, tz, 7)
    assert _tiles(n, lat.tile()) <= MOST_TILES
    lat.set_stencil("27")
    say("tz", tz, "27-point shape", lat.tile(), "tiles", _tiles(n, lat.tile()))
    assert _tiles(n, lat.tile()) <= MOST_TILES
    if tz == 16:                                  # few enough: the length stays
        assert lat.tile()[3] == 16
    lat.close()


def test_tuned_chunk_is_not_a_given_one():
    """What a tuner found for the 7-point pass (the batch tuner's chunks have at
    least four planes) says nothing of the 27-point one: after the change the
    shape is that of a lattice never tuned, at 48^3 one plane a chunk."""
    def fresh():
        lat = sl.Lattice(48, 2, 20.0, precision="f32")
        lat.set_potential("chaotic2", (1.0, 10.0))
        return lat
    want = fresh()
    want.set_stencil("27")
    lat = fresh()
    lat.init_fluctuations((0.5, 0.0), (0.0, 0.0), "white", 1e-3, 3)
    b = sl.Batch()
    b.add(lat)
    b.autotune(reps=1)
    tuned = lat.tile()
    b.remove(lat)
    b.close()
    lat.set_stencil("27")
    say("tuned", tuned, "27-point", lat.tile(), "never tuned", want.tile())
    assert tuned[3] >= 4 and lat.tile() == want.tile()
    lat.close()
    want.close()


def test_first_batch_member_keeps_its_given_chunk():
    """128^3, one FP32 field: the shape of the 7-point pass is the default (four
    sites per lane) but for its chunk length; the first member brings two sites
    per lane into a batch, which more sides can share, and the same chunk."""
    lat = sl.Lattice(128, 1, 20.0, precision="f32")
    lat.set_potential("free", (1.0,))
    lat.set_stencil("27")
    lat.set_tile(16, 1, 12, 1)
    lat.set_stencil("7")
    assert lat.tile()[1] == 4 and lat.tile()[3] == 12
    lat.init_fluctuations((0.5,), (0.0,), "white", 1e-3, 3)
    other = sl.Lattice(66, 1, 20.0, precision="f32")
    other.set_potential("free", (1.0,))
    other.init_fluctuations((0.5,), (0.0,), "white", 1e-3, 4)
    b = sl.Batch()
    b.add(lat)
    b.add(other)
    say("member", lat.tile(), "second", other.tile())
    assert lat.tile()[1] == 2 and lat.tile()[3] == 12 and other.tile()[1] == 2
    b.step(2, 0.005, 4)
    b.close()
    lat.close()
    other.close()
