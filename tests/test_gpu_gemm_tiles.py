"""The tiled FP64 product at the edges of its tiles and slabs, in both forms of
its operand loads: 16 bytes a lane (even base, leading dimension and extent, or
a padded odd extent) and 4 bytes a lane (everything else)."""
import pytest
import torch

from paper_1805_08990_amd import _binding as b
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


def _block(rows, cols, pad, off, gen):
    """A rows x cols block at leading dimension rows + pad, off doubles into its
    buffer, whose last column is the buffer's end; NaN around it."""
    ld = rows + pad
    buf = torch.full((off + ld * (cols - 1) + rows,), float("nan"), dtype=torch.float64, device="cuda")
    blk = buf.as_strided((rows, cols), (1, ld), off)
    blk.copy_(torch.randn(rows, cols, generator=gen, dtype=torch.float64, device="cuda"))
    return buf, blk, ld


# 64 x 64, 128 x 64 and 128 x 128 tiles; depths of less than a slab, whole
# slabs, one more, and enough for a split
SIZES = [(257, 300, 5), (300, 257, 16), (320, 384, 48), (259, 513, 33), (385, 258, 2100),
         (2047, 1100, 31), (2048, 1088, 64), (2050, 2049, 17), (2049, 2050, 80)]


@pytest.mark.parametrize("M,N,K", SIZES)
@pytest.mark.parametrize("trans", ["NN", "TN", "NT", "TT"])
@pytest.mark.parametrize("pad,off", [(0, 0), (1, 0), (2, 2), (2, 1)])
def test_gemm_tiles(ctx, M, N, K, trans, pad, off):
    announce("gemm tiles", M, N, K, trans, pad, off)
    gen = torch.Generator("cuda").manual_seed(M + 3 * N + 7 * K + pad)
    ab, A, lda = _block(*((M, K) if trans[0] == "N" else (K, M)), pad, off, gen)
    bb, B, ldb = _block(*((K, N) if trans[1] == "N" else (N, K)), pad, off, gen)
    cb, C, ldc = _block(M, N, pad, off, gen)
    opA, opB = (A if trans[0] == "N" else A.t()), (B if trans[1] == "N" else B.t())
    ref = 0.75 * (opA @ opB) - 0.5 * C
    # the dot product's error bound on each side, K units of roundoff on |A||B|
    scale = 0.75 * (opA.abs() @ opB.abs()) + 0.5 * C.abs()
    rc = b._lib_gemm(ctx._h, trans[0].encode(), trans[1].encode(), M, N, K, 0.75, A.data_ptr(), lda,
                     B.data_ptr(), ldb, -0.5, C.data_ptr(), ldc)
    torch.cuda.synchronize()
    assert rc == b.DME_OK
    assert bool(((C - ref).abs() <= 2 * (K + 2) * 2.3e-16 * scale).all())
    # nothing around the block was written
    mask = torch.ones_like(cb, dtype=torch.bool)
    mask.as_strided((M, N), (1, ldc), off).fill_(False)
    assert bool(cb[mask].isnan().all())
