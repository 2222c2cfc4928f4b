"""The stored linearisation rows of one coordinated-turn target leave out what a
regression reproduces exactly (the turn rate's row of F, c and Q', the columns of
H that a bearing does not read).  Checked with a process noise that couples the
turn rate to every other state, so that row 4 of Q' is not the usual diagonal
one, at lane and tile edges, on every path that reads the rows: the scans in both
forms, the sequential path and the filtering pass with its likelihood.  Against
the oracle, which stores every row, at the FP64 gate of the other parity tests
(one iteration from a common start)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2102_00514_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL = 1e-9


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2102_00514_amd import binding
    return binding


def _coupled(T):
    pb = wl.ct_bearings(T, seed=700 + T)
    d = np.sqrt(np.diag(pb.Q))
    corr = 0.25 * np.ones((5, 5)) + 0.75 * np.eye(5)
    corr[4, :4] = corr[:4, 4] = (0.1, -0.2, 0.3, 0.15)
    return dataclasses.replace(pb, Q=d[:, None] * corr * d[None, :])


@pytest.mark.parametrize("T", (1, 2, 63, 64, 257))
@pytest.mark.parametrize("lin", ("cubature", "unscented"))
@pytest.mark.parametrize("kw", (dict(), dict(lane_slots=4), dict(scan="sequential"), dict(form="sqrt")),
                         ids=("scan", "slots4", "sequential", "sqrt"))
def test_smoother(B, T, lin, kw):
    pb = _coupled(T)
    ref = oracle.smoother(pb, 1, lin)
    with B.Smoother(pb, n_iter=1, lin=lin, **kw) as sm:
        sm.iterate(1, want_delta=False)
        mean, cov = sm.result()
    assert oracle.mean_error(mean, ref["mean"]) < TOL
    assert oracle.cov_error(cov, ref["cov"]) < TOL


@pytest.mark.parametrize("T", (1, 64, 300))
def test_filter(B, T):
    pb = _coupled(T)
    ref = oracle.filter_loglik(pb, "cubature")
    with B.Smoother(pb, n_iter=1, lin="cubature") as sm:
        mean, cov, ll = sm.filter()
    assert oracle.mean_error(mean, ref["filt_mean"]) < TOL
    assert oracle.cov_error(cov, ref["filt_cov"]) < TOL
    assert abs(ll[0] - ref["loglik"]) <= TOL * max(abs(ref["loglik"]), 1.0)
