"""Eigenpairs of small symmetric matrices at the edges of the register-resident
formation of Q (k <= 64, 128, 192, chunks of 16 reflectors, four columns a
block) and of the division-free Sturm counts (scaling, exactly decoupled and
repeated entries), against numpy's eigenvalues in float64.

The reduction and the counts are backward stable, so eigenvalues are within a
few k eps ||M|| (1e-13 sqrt(k) ||M|| is above that for k <= 192); vectors and
residual are held to 1e-12 sqrt(k), as for any other size.
"""
import numpy as np
import pytest

from tests.gpu_common import announce, to_np

pytestmark = pytest.mark.gpu


def _matrix(kind, k):
    rng = np.random.default_rng(7 * k + len(kind))
    X = rng.standard_normal((k, k))
    M = 0.5 * (X + X.T)
    if kind == "small":
        return M * 2.0 ** -100
    if kind == "large":
        return M * 2.0 ** 100
    if kind == "diag":  # every off-diagonal entry exactly zero, values repeated
        return np.diag(np.round(3.0 * rng.standard_normal(k)) + 0.5)
    if kind == "blocks":  # decoupled, one block far below the other
        M[: k // 2, k // 2:] = 0.0
        M[k // 2:, : k // 2] = 0.0
        M[: k // 2, : k // 2] *= 2.0 ** -30
    return M


@pytest.mark.parametrize("kind", ["plain", "small", "large", "diag", "blocks"])
@pytest.mark.parametrize("k", [2, 3, 4, 9, 18, 19, 65, 130, 192])
def test_eigenpairs(ctx, kind, k):
    announce("eigenpairs", kind, k)
    M = _matrix(kind, k)
    lam, V, kk = ctx.syev(M, tol=1e-17)
    lam, V = to_np(lam), to_np(V)
    ref = np.linalg.eigvalsh(M)
    assert kk == k
    assert np.max(np.abs(np.sort(lam) - ref)) <= 1e-13 * np.sqrt(k) * np.abs(ref).max()
    assert np.linalg.norm((V * lam) @ V.T - M) <= 1e-12 * np.linalg.norm(M) * np.sqrt(k)
    assert np.max(np.abs(V.T @ V - np.eye(k))) <= 1e-12 * np.sqrt(k)
