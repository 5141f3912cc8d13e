"""Eigenpairs do not depend on what the context's workspace held: a split product
of NaN matrices fills it with NaN first.  The matrices have columns that need no
reflector (exactly zero below the subdiagonal), whose place the reduction leaves
unwritten: diagonal, decoupled blocks, and zero but for a corner."""
import numpy as np
import pytest
import torch

from tests.gpu_common import announce, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nan_operand():
    return torch.full((256, 65536), float("nan"), dtype=torch.float64, device="cuda")


def _matrix(kind, k):
    rng = np.random.default_rng(3 * k + len(kind))
    X = rng.standard_normal((k, k))
    M = 0.5 * (X + X.T)
    if kind == "diag":
        return np.diag(np.round(3.0 * rng.standard_normal(k)) + 0.5)
    if kind == "blocks":
        h = k // 2
        M[:h, h:] = 0.0
        M[h:, :h] = 0.0
        return M
    M[k // 3 + 1:, :] = 0.0  # corner
    M[:, k // 3 + 1:] = 0.0
    return M


@pytest.mark.parametrize("kind", ["diag", "blocks", "corner"])
@pytest.mark.parametrize("k", [3, 16, 17, 64, 65, 128, 150, 192, 300])
def test_workspace_contents(ctx, nan_operand, kind, k):
    announce("eigenpairs after NaN in the workspace", kind, k)
    M = _matrix(kind, k)
    ctx.syev(np.eye(300), tol=0.5)  # the workspace as large as any size here needs
    # 256 x 256 with K split: the partial sums, NaN, cover the workspace's first megabytes
    C = ctx.gemm(nan_operand, nan_operand, transb="T")
    lam, V, kept = ctx.syev(M, tol=1e-12)
    assert bool(torch.isnan(C).all())
    lam, V = to_np(lam)[:kept], to_np(V)
    ref = np.linalg.eigvalsh(M)
    top = np.abs(ref).max()
    assert kept == int(np.sum(np.abs(ref) > 1e-12 * top))
    assert np.linalg.norm((V * lam) @ V.T - M) <= 1e-12 * np.linalg.norm(M) * np.sqrt(k)
    assert np.max(np.abs(V.T @ V - np.eye(kept))) <= 1e-12 * np.sqrt(k)
