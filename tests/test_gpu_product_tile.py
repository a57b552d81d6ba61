"""GPU parity of int8 products on more 64 x 64 tiles than the chip holds at once, over the codes that the choice among them
has: the 128 x 256 tile with no K tile, one, fewer than its stages and many, last rows and columns of a tile that are
missing, every bias layout, several tiles to a workgroup; bit for bit.  test_gemm_rules.py holds each shape to its kernel."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu


TILE_128X256 = [
    (1108, 6544, 32), (1105, 6672, 16), (3659, 1216, 192), (3264, 1296, 400), (3302, 1296, 496), (5788, 960, 208),
    (1656, 2624, 1040), (2100, 2100 // 16 * 16, 80), (1100, 6544, 0)]
SEVERAL_TO_A_WORKGROUP = [(3147, 7440, 16), (4990, 4336, 96), (668, 23056, 208)]  # more of them than the 512 that the chip holds
OTHER_CODES = [(5050, 3600, 176), (5676, 640, 512)]  # weight-stationary where the bias is a row, 128 x 128


@pytest.mark.parametrize("kind", ["row", "none", "matrix"])
@pytest.mark.parametrize("M,N,K", TILE_128X256 + SEVERAL_TO_A_WORKGROUP + OTHER_CODES)
def test_products(M, N, K, kind):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + N + K, bias_matrix=kind == "matrix")
    t = None if kind == "none" else dev(b)
    if kind == "none":
        b = np.zeros_like(b)
    C = torch.full((M, N), 9, dtype=torch.int8, device="cuda")
    At, Bt = (dev(A), dev(B)) if K else (torch.zeros((M, 16), dtype=torch.int8, device="cuda")[:, :0], torch.zeros((16, N), dtype=torch.int8, device="cuda")[:0])
    ops.ac_gemm_i8(At, Bt, t, C, 8, 1)
    np.testing.assert_array_equal(host(C), oracle.gemm_i8(A, B, b, 8, 1))
