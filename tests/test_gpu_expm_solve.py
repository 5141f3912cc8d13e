"""The Pade denominator's solve inside dme_expm, where its factorisation can go
wrong: operators whose denominator needs row exchanges (rotations by about a
half turn leave a nearly zero diagonal), at the edges of its 32-column panels,
64-column blocks and 512-row tournament groups."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import announce, rel_fro, to_np

pytestmark = pytest.mark.gpu

# dme_expm's parity bar: the denominator's condition number is below
# e^theta_13 ~ 220, so a backward stable solve stays far inside it
TOL = 1e-12


@pytest.mark.parametrize("n", [1, 2, 31, 33, 63, 64, 65, 96, 97, 129, 512, 513, 545, 1100])
def test_expm_dense_rotation(ctx, n):
    announce("expm rotation", n)
    rng = np.random.default_rng(n)
    G = rng.standard_normal((n, n))
    X = G - G.T + 0.05 * G
    X *= 5.0 / max(oracle.norm1(X), 1e-300)  # [13/13], no squaring
    E, m, s = ctx.expm(X, 1.0)
    assert (m, s) == (oracle.expm_params(oracle.norm1(X)))
    assert rel_fro(to_np(E), oracle.expm(X)) < TOL


@pytest.mark.parametrize("n,theta", [(1000, 3.141592653589793), (2050, 3.0), (8300, 3.141592653589793)])
def test_expm_permuted_plane_rotations(ctx, n, theta):
    """Plane rotations under a random symmetric permutation: e^X is known, the
    pivots are far from the diagonal, and 8300 rows take three tournament
    levels."""
    announce("expm plane rotations", n, theta)
    perm = torch.from_numpy(np.random.default_rng(n).permutation(n)).cuda()
    i, j = perm[: n // 2], perm[n // 2: 2 * (n // 2)]
    X = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    X[i, j] = theta
    X[j, i] = -theta
    E, m, s = ctx.expm(X, 1.0)
    ref = torch.zeros_like(X)
    ref.fill_diagonal_(1.0)
    ref[i, i] = np.cos(theta)
    ref[j, j] = np.cos(theta)
    ref[i, j] = np.sin(theta)
    ref[j, i] = -np.sin(theta)
    assert (m, s) == (13, 0)
    assert float((E - ref).norm() / ref.norm()) < TOL


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 257, 300, 513, 1030, 2049])
@pytest.mark.parametrize("nrm", [5.0, 50.0])
def test_expm_symmetric(ctx, n, nrm):
    """An exactly symmetric operator: half products and the positive definite
    denominator's inverse, at the edges of 64-row blocks and of the tiles."""
    announce("expm symmetric", n, nrm)
    G = np.random.default_rng(n).standard_normal((n, n))
    X = G + G.T
    X *= nrm / max(oracle.norm1(X), 1e-300) * (1.0 - 1e-12)
    X = (X + X.T) / 2
    E, m, s = ctx.expm(X, 1.0)
    assert (m, s) == (oracle.expm_params(oracle.norm1(X)))
    E = to_np(E)
    assert rel_fro(E, oracle.expm(X)) < TOL
    if n > 256:
        assert np.array_equal(E, E.T)
