"""The nx = 20 engine's Cholesky factorisation and substitutions (n = 20 and
the n = 8 of the measurements, FP64 and FP32) at the edges of the fast form:
pivots inside 2^-664 .. 2^664, just outside (the form with the library root
and division), and matrices that are not positive definite.  Tolerances: the
backward error of a Cholesky factorisation and of a triangular solve is below n
units of rounding of the matrix norm; 4 n units allow for the condition number
(below 100) in the solutions."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _spd(rng, n, count):
    Q = np.linalg.qr(rng.standard_normal((count, n, n)))[0]
    ev = np.exp(rng.uniform(np.log(0.02), 0.0, (count, n)))
    A = (Q * ev[:, None, :]) @ Q.transpose(0, 2, 1)
    return 0.5 * (A + A.transpose(0, 2, 1))


@pytest.mark.parametrize("n, dtype, scale", [
    (20, "float64", 1.0), (20, "float64", 2.0 ** -650), (20, "float64", 2.0 ** -670), (20, "float64", 2.0 ** 662),
    (20, "float64", 2.0 ** 700), (20, "float32", 1.0), (20, "float32", 2.0 ** -110), (20, "float32", 2.0 ** 110),
    (8, "float64", 1.0), (8, "float64", 2.0 ** -700), (8, "float32", 1.0)])
def test_factor_and_solves(n, dtype, scale):
    import torch
    from paper_2102_00514_amd import dense_probe as dp
    rng = np.random.default_rng(n)
    A = _spd(rng, n, 70).astype(dtype)
    X = rng.standard_normal(A.shape).astype(dtype)
    root = np.sqrt(scale)                       # a power of two: scaling is exact
    dA, dX = torch.from_numpy((A * A.dtype.type(scale))).cuda(), torch.from_numpy(X).cuda()
    L, Y, Z, ok = (v.cpu().numpy() for v in dp.factor(dp.load(), dA, dX, torch.cuda.current_stream().cuda_stream))
    assert np.all(ok == 1)
    assert np.all(np.triu(L, 1) == 0.0)
    eps = np.finfo(dtype).eps
    L64, A64, X64 = L.astype(np.float64) / root, A.astype(np.float64), X.astype(np.float64)
    tol = 4 * n * eps
    assert np.abs(L64 @ L64.transpose(0, 2, 1) - A64).max() < tol
    Y64, Z64 = Y.astype(np.float64) * root, Z.astype(np.float64) * scale
    assert np.abs(L64 @ Y64 - X64).max() < tol * np.abs(L64).max() * np.abs(Y64).max()
    assert np.abs(L64.transpose(0, 2, 1) @ Z64 - Y64).max() < tol * np.abs(L64).max() * np.abs(Z64).max()


@pytest.mark.parametrize("n", [20, 8])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_not_positive_definite_is_flagged(n, dtype):
    import torch
    from paper_2102_00514_amd import dense_probe as dp
    rng = np.random.default_rng(3)
    A = _spd(rng, n, 6).astype(dtype)
    A[1, 0, 0] = -1.0                            # first pivot
    A[2, n - 1, n - 1] = -3.0                    # last pivot
    A[3, n // 2, n // 2] = np.nan
    A[4] = 0.0
    dA, dX = torch.from_numpy(A).cuda(), torch.from_numpy(np.ones_like(A)).cuda()
    L, Y, _, ok = (v.cpu().numpy() for v in dp.factor(dp.load(), dA, dX, torch.cuda.current_stream().cuda_stream))
    assert ok.tolist() == [1, 0, 0, 0, 0, 1]
    for b in (1, 2, 3):
        assert not np.all(np.isfinite(L[b]))     # reaches the convergence statistic
    assert np.all(np.isfinite(L[[0, 5]])) and np.all(np.isfinite(Y[[0, 5]]))
