"""The quadrature nodes' exponentials of a nonsymmetric operator, whose LU
solves run together: sizes at the edges of the 32-column panels, the 64-column
blocks and the 192-row leaves of the pivot tournament, odd sizes (padded leading
dimension), and node times whose exponentials take different degrees and numbers
of squarings."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from paper_1805_08990_amd import _binding as b
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 31, 33, 64, 65, 97, 193, 258])
@pytest.mark.parametrize("size", [0.05, 60.0])  # ||A||_1: all of low degree; degrees 3 to 13 with squarings
def test_node_exponentials(ctx, n, size):
    announce("node exponentials", n, size)
    G = wl.random_nonsymmetric(n, seed=n)
    A = G - 1.2 * np.linalg.norm(G, 2) * np.eye(n)
    A *= size / np.linalg.norm(A, 1)
    C = wl.random_C(2, n, 5)
    h, steps = 0.2, 2
    L, D, k = ctx.solve("dle", b.SolveOptions(T=steps * h, h=h, tol=1e-12, precision="fp64"), A, C)
    Lo, Do, _ = oracle.solve(A, C, steps * h, h, kind="dle", tol=1e-12)
    assert k == steps
    assert oracle.lowrank_rel_err(L, D, Lo, Do) < 1e-10


# a few tiles more than whole rounds of the chip (32 to 35 tiles of 128 a side),
# the last one whole, ragged at either quarter, and a single row
@pytest.mark.parametrize("n", [4096, 4033, 4000, 4097, 4421])
def test_symmetric_products_with_few_tiles_left(ctx, n):
    """e^X of the 1D Laplacian, whose eigenvectors are sines."""
    announce("symmetric tail", n)
    i = torch.arange(1, n + 1, dtype=torch.float64, device="cuda")
    S = np.sqrt(2.0 / (n + 1)) * torch.sin(np.pi / (n + 1) * (i[:, None] * i[None, :] % (2 * (n + 1))))
    lam = -3.0 * (2.0 - 2.0 * torch.cos(np.pi / (n + 1) * i))  # ||X||_1 = 12: [13/13], two squarings
    X = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    X.diagonal().fill_(-6.0)
    X.diagonal(1).fill_(3.0)
    X.diagonal(-1).fill_(3.0)
    E, m, s = ctx.expm(X, 1.0)
    assert (m, s) == (13, 2)
    ref = (S * torch.exp(lam)) @ S
    assert float(torch.linalg.norm(E - ref) / torch.linalg.norm(ref)) < 1e-12
    assert torch.equal(E, E.t())
