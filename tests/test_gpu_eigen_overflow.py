"""A symmetric matrix of finite entries whose Householder reduction overflows: the
first row of the tridiagonal matrix is finite, the rest is not, so no twist index
compares.  The eigenvalue call ends like any other (there is nothing to check in
what it gives for such a matrix), and the next one is right."""
import numpy as np
import pytest

from tests.gpu_common import announce, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [3, 40, 64, 96, 128, 150, 180, 300])
def test_overflowing_reduction(ctx, k):
    announce("eigen overflow", k)
    rng = np.random.default_rng(k)
    X = rng.standard_normal((k, k))
    M = 0.5 * (X + X.T)
    big = M.copy()
    big[1:, 1:] *= 1e200  # squares past the largest double from the second column on
    lam, V, kept = ctx.syev(big, tol=1e-17)
    assert 0 <= kept <= k

    lam, V, kept = ctx.syev(M, tol=1e-17)
    lam, V = to_np(lam), to_np(V)
    ref = np.linalg.eigvalsh(M)
    assert kept == k
    assert np.max(np.abs(np.sort(lam) - ref)) <= 1e-13 * np.sqrt(k) * np.abs(ref).max()
    assert np.max(np.abs(V.T @ V - np.eye(k))) <= 1e-12 * np.sqrt(k)
