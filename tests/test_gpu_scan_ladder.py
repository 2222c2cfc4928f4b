"""The scan ladders at the edges of their wavefronts: tiles whose last wavefronts
hold few real slots or none, two and four wavefronts joined, one to three tiles,
and tile aggregates that fill the single-block scan's first wavefront exactly or
by one more.  The parallel scans are compared with the sequential ones.

Both evaluate the same smoother in FP64 from the same starting trajectory; a
scan of S slots accumulates at most S roundings, amplified by the ratio of the
largest to the smallest covariance entry (1e4 here): 513 * 2.2e-16 * 1e4 = 1.1e-9
relative to the largest value of a component.  Past a few hundred slots the
smoother has forgotten a rounding, so the bound holds for the long tracks too."""
import numpy as np
import pytest

from paper_2102_00514_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL = 513 * 2.0 ** -52 * 1e4
LENGTHS = (1, 15, 16, 31, 32, 62, 63, 64, 127, 128, 191, 192, 255, 256, 300, 512, 64 * 256, 65 * 256)


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2102_00514_amd import binding
    return binding


def _run(B, pb, **kw):
    with B.Smoother(pb, n_iter=2, **kw) as sm:
        sm.iterate(2, want_delta=False)
        return sm.result()


def _compare(B, pb, **kw):
    m, c = _run(B, pb, **kw)
    ms, cs = _run(B, pb, scan="sequential", **kw)
    for got, want in ((m, ms), (c.reshape(len(m), -1), cs.reshape(len(m), -1))):
        scale = np.abs(want).max(axis=0)
        assert np.all(np.abs(got - want) <= TOL * scale)


@pytest.mark.parametrize("T", LENGTHS)
def test_one_track(B, T):
    _compare(B, wl.ct_bearings(T, seed=300 + T), lin="taylor")


@pytest.mark.parametrize("last", (1, 63, 64, 130))
def test_batch(B, last):
    tracks = [wl.ct_bearings(T, seed=400 + T) for T in (250, 3, 70, last)]
    _compare(B, wl.concat_tracks(tracks, "ladder"), lin="cubature")


@pytest.mark.parametrize("tiles", (512, 513, 2048, 2049))
@pytest.mark.parametrize("limit", (0, 1 << 33), ids=("free", "limited"))
def test_many_tiles(B, tiles, limit):
    """One block over the tile aggregates, or levels of 64-lane blocks: 512 tiles
    without a memory limit and 2048 with one are the last that one block scans."""
    base = [wl.ct_bearings(499, seed=800 + i) for i in range(3)]
    slots = tiles * 64 - 5
    n = slots // 500
    tracks = [base[i % 3] for i in range(n)]
    if slots - 500 * n > 1:
        tracks.append(wl.ct_bearings(slots - 500 * n - 1, seed=900))
    pb = wl.concat_tracks(tracks, "tiles")
    with B.Smoother(pb, n_iter=1, tile_lanes=64, lane_slots=1, max_device_bytes=limit) as sm:
        assert sm.schedule()[2] == tiles
    _compare(B, pb, lin="taylor", tile_lanes=64, lane_slots=1, max_device_bytes=limit)


@pytest.mark.parametrize("T", (1, 15, 16, 17, 62, 63, 64, 127, 300, 64 * 64, 64 * 256, 64 * 257))
def test_square_root_form(B, T):
    """The square-root operator on elements in LDS: edges of rows and wavefronts,
    and top scans of one slot a lane (256 tiles) and of two (257)."""
    pb = wl.ct_bearings(T, seed=1000 + T)
    m, c = _run(B, pb, lin="taylor", form="sqrt")
    ms, cs = _run(B, pb, lin="taylor")
    for got, want in ((m, ms), (c.reshape(len(m), -1), cs.reshape(len(m), -1))):
        scale = np.abs(want).max(axis=0)
        assert np.all(np.abs(got - want) <= TOL * scale)


@pytest.mark.parametrize("nx, tiles", [(5, 768), (5, 769), (3, 1024), (3, 1025), (1, 1792), (1, 1793)])
def test_last_tiles_of_one_block(B, nx, tiles):
    """The last number of tiles that one block scans without a memory limit, and
    the first that goes through levels, by the size of the state."""
    T = tiles * 64 - 9
    pb = wl.ct_bearings(T, seed=nx) if nx == 5 else wl.linear_gaussian(nx, {1: 1, 3: 2}[nx], T, seed=nx)
    with B.Smoother(pb, n_iter=1, lin="taylor", tile_lanes=64, lane_slots=1) as sm:
        assert sm.schedule()[2] == tiles
    _compare(B, pb, lin="taylor", tile_lanes=64, lane_slots=1)


@pytest.mark.parametrize("slots", (2, 4))
@pytest.mark.parametrize("T", (3, 130, 256, 700, 256 * 4 * 3 - 2))
def test_exclusive_prefixes_of_four_wavefronts(B, slots, T):
    """Several slots a lane: the lanes' exclusive prefixes across wavefronts, last
    wavefronts that hold padding among them."""
    _compare(B, wl.ct_bearings(T, seed=500 + T), lin="taylor", tile_lanes=256, lane_slots=slots)
