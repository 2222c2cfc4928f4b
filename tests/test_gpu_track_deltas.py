"""Per-track change statistics of tiles that hold several tracks, at the edges
of the table in which a tile gathers them: exactly the largest change of the
returned means (both are FP64 differences of the same stored values)."""
import numpy as np
import pytest

from paper_2102_00514_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes, slots, lengths", [
    (256, 4, [1] * 200),                      # more tracks in a tile than table entries
    (64, 2, [1] * 63 + [2]),                  # 64 tracks over the first tile and into the next
    (64, 16, [3, 1500, 1, 1, 700, 2, 40]),    # runs that start and end inside a lane
    (256, 1, [255, 1, 300, 7, 7, 7]),
    (64, 4, [5000]),                          # one track
])
def test_track_deltas_are_the_changes_of_the_means(lanes, slots, lengths):
    from paper_2102_00514_amd import binding
    parts = [wl.ct_bearings(T, seed=i) for i, T in enumerate(lengths)]
    pb = wl.concat_tracks(parts)
    with binding.Smoother(pb, n_iter=3, lin="taylor", tile_lanes=lanes, lane_slots=slots) as sm:
        sm.iterate(1)
        before, _ = sm.result()
        sm.iterate(1)
        after, _ = sm.result()
        deltas = sm.track_deltas()
    so = pb.slot_offsets()
    want = [np.abs(after[so[i]:so[i + 1]] - before[so[i]:so[i + 1]]).max() for i in range(pb.n_tracks)]
    np.testing.assert_array_equal(deltas, want)
