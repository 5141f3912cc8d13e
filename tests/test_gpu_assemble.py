"""A compression's input assembled in one launch ([L, C^T] and blkdiag(D, t I)
in the split with T1 and T2, the quadrature factor's columns and blkdiag(D, D_I)
otherwise): fewer rows than columns, and rows past one and two blocks of 1024."""
import pytest

import oracle
import workloads as wl
from paper_1805_08990_amd import _binding as b
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", ["F1F2", "F12"])
@pytest.mark.parametrize("nx,p", [(2, 4), (3, 7), (32, 3), (33, 2), (46, 1)])
def test_assembled_input(ctx, split, nx, p):
    announce("assemble", split, nx, p)
    n, h, steps = nx * nx, 1e-3, 3
    A, C = wl.laplacian_2d(nx), wl.random_C(p, n, nx)
    L, D, k = ctx.solve("dle", b.SolveOptions(T=steps * h, h=h, tol=1e-10, split=split, precision="fp64"), A, C)
    Lo, Do, _ = oracle.solve(A, C, steps * h, h, kind="dle", tol=1e-10, split=split)
    assert k == steps
    assert oracle.lowrank_rel_err(L, D, Lo, Do) < 1e-10
