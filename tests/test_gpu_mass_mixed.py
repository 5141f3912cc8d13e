"""The mass matrix of a mixed-precision solve is factored with a division for
every multiplier, as all of what feeds the split-BF16 products: for
M^T = [[49 I, c I], [49 I, (c + 1) I]] with a large c the multipliers are exactly
one and the solution is exact, while 49 (1 / 49) < 1 would leave c times that
difference in it.  The rows of a pair lie in different panels of the
factorisation, and the standard form A M^-1, C M^-1 is known in advance."""
import numpy as np
import pytest

import oracle
import workloads as wl
from paper_1805_08990_amd import _binding as b
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [80, 128, 190])
def test_mixed_mass_matrix_divides(ctx, n):
    announce("mixed mass matrix", n)
    q, c = n // 2, 2.0 ** 44
    eye = np.eye(q)
    Mt = np.block([[49.0 * eye, c * eye], [49.0 * eye, (c + 1.0) * eye]])
    rng = np.random.default_rng(n)
    # multiples of 1/8 whose products with 49 are exact; no dependence on the second half
    Xa = np.zeros((n, n))
    Xa[:q] = np.round(8.0 * rng.standard_normal((q, n))) / 64.0
    Xa[:q, :q] -= 16.0 * eye
    Xc = np.zeros((n, 2))
    Xc[:q] = np.round(8.0 * wl.random_C(2, q, n).T) / 8.0 + 0.125
    A, C = (Mt @ Xa).T, (Mt @ Xc).T
    h, steps = 0.01, 4
    L, D, k = ctx.solve("dle", b.SolveOptions(T=steps * h, h=h, tol=1e-10, precision="mixed"), A, C, M=Mt.T)
    Lo, Do, _ = oracle.solve(Xa.T, Xc.T, steps * h, h, kind="dle", tol=1e-10)
    assert k == steps
    assert oracle.lowrank_rel_err(L, D, Lo, Do) < 1e-6  # the mixed mode's bar
