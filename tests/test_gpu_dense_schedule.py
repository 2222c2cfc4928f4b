"""The nx = 20 engine's own choice of slots per wave, at the edges of its rule:
the schedule it reports, and the same result as with eight slots per wave (the
scan trees differ, so to rounding: the FP64 parity gate)."""
import numpy as np
import pytest

import oracle
from paper_2102_00514_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots, precision, cap, want", [
    (2, "f64", 0, 2), (501, "f32", 0, 8), (3072, "f64", 0, 2), (3073, "f64", 0, 4), (12288, "f64", 0, 4),
    (12289, "f64", 0, 8), (501, "f64", 1 << 34, 8)])
def test_automatic_slots_per_wave(slots, precision, cap, want):
    from paper_2102_00514_amd import binding
    pb = wl.stacked_ct(slots - 1, np.random.default_rng([5, 90]))
    out = []
    for k in (0, 8):
        with binding.Smoother(pb, n_iter=1, lin="unscented", precision=precision, lane_slots=k,
                              max_device_bytes=cap) as sm:
            if k == 0:
                assert sm.schedule()[1] == want
            sm.iterate(1)
            out.append(sm.result())
    assert oracle.mean_error(out[0][0], out[1][0]) < 1e-9
    assert oracle.cov_error(out[0][1], out[1][1]) < 1e-9
