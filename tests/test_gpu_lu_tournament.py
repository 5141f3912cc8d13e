"""The LU of a Pade denominator where its pivot tournament gains a level: up
to 192 rows are one wave's, and the 32 rows that each of six waves names (6 x 192 =
1152 rows) are one wave's again.  The operators are rotations by about a half turn, whose
denominator needs row exchanges; its condition number is below e^theta_13 ~ 220,
so a backward stable solve stays far inside 1e-12."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import announce, rel_fro, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [191, 192, 193, 256, 1152, 1153])
def test_tournament_levels(ctx, n):
    announce("LU tournament", n)
    rng = np.random.default_rng(n)
    G = rng.standard_normal((n, n))
    X = G - G.T + 0.05 * G
    X *= 5.0 / oracle.norm1(X)  # [13/13], no squaring
    E, m, s = ctx.expm(X, 1.0)
    assert (m, s) == oracle.expm_params(oracle.norm1(X))
    assert rel_fro(to_np(E), oracle.expm(X)) < 1e-12
