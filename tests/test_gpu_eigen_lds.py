"""Eigenpairs do not depend on what earlier kernels left in LDS: a product of NaN
matrices fills the LDS of every CU with NaN first.  Sizes over every tile shape of
the register-resident reduction, and all of the range (k = 129 .. 160) whose rows
are not whole waves of lanes."""
import numpy as np
import pytest
import torch

from tests.gpu_common import announce, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nan_operand():
    return torch.full((4096, 64), float("nan"), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("k", [2, 33, 64, 65, 128, 129, 136, 137, 144, 150, 159, 160, 161, 192])
def test_lds_contents(ctx, nan_operand, k):
    announce("eigenpairs after NaN in LDS", k)
    rng = np.random.default_rng(k)
    X = rng.standard_normal((k, k))
    M = 0.5 * (X + X.T)
    # 32 x 32 tiles of 128 x 128, two to a CU, each with 64 KiB of its operands in LDS
    C = ctx.gemm(nan_operand, nan_operand, transb="T")
    lam, V, kept = ctx.syev(M, tol=1e-17)
    assert bool(torch.isnan(C).all())
    lam, V = to_np(lam), to_np(V)
    ref = np.linalg.eigvalsh(M)
    assert kept == k
    # backward stable: a few k eps ||M||, and vectors orthonormal by the polar steps
    assert np.max(np.abs(np.sort(lam) - ref)) <= 1e-13 * np.sqrt(k) * np.abs(ref).max()
    assert np.linalg.norm((V * lam) @ V.T - M) <= 1e-12 * np.linalg.norm(M) * np.sqrt(k)
    assert np.max(np.abs(V.T @ V - np.eye(k))) <= 1e-12 * np.sqrt(k)
