"""The forms of the product kernels that are chosen by size, at the sizes where each can go wrong."""
import numpy as np
import pytest
import torch

from oracle import mx_oracle as orc
from paper_2307_15517_amd import mx
from test_gpu_parity import check_product, gpu_operand, host, random_operand

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,block,wa,wb", [
    (9, 32, 64, 16, 8, 4),             # one chunk of K: fifteen of the sixteen waves have none
    (16, 40, 17 * 64, 16, 8, 4),       # the tile's upper rows do not exist; one wave has a second chunk
    (17, 33, 48, 16, 5, 7),            # one row in the upper half, a partial chunk
    (33, 1, 9 * 128, 32, 6, 5),        # one column, eight waves and one chunk more
    (64, 64, 3 * 256, 64, 8, 8),
    (40, 32 * 270, 128, 16, 8, 4),     # 540 tiles: eight waves each
    (70, 32 * 350 + 5, 64, 16, 4, 4),  # 1053 tiles: four waves each
])
def test_fragment_product_tiles_and_waves(M, N, K, block, wa, wb):
    """Block exponents on both sides of the range in which the scales are built by an integer instruction (bytes 96 to
    159), the other way for whole operands, and zero blocks (byte 0) among ordinary ones."""
    rng = np.random.default_rng(M * N + K)
    for lo, hi in ((96, 160), (94, 99), (157, 162)):
        qa, ea = random_operand(rng, M, K, block, wa, lo, hi)
        qb, eb = random_operand(rng, N, K, block, wb, 100, 150)
        zero = rng.random(ea.shape) < 0.1
        ea[zero] = 0
        qa.reshape(M, K // block, block)[zero] = 0
        A, fa = gpu_operand(qa, ea, block, wa)
        B, fb = gpu_operand(qb, eb, block, wb)
        y = mx.gemm(A, fa, B, fb, M, N, K)
        torch.cuda.synchronize()
        y_ref, mag = orc.gemm(qa, ea, wa, qb, eb, wb, block, want_mag=True)
        check_product(host(y)[0], y_ref, mag, "%dx%dx%d bytes %d..%d" % (M, N, K, lo, hi - 1))
