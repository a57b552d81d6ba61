"""GPU parity of the 4-byte output stages of the direct-to-LDS tiles where they read beside the product: int32 with a bias row, a bias
matrix and none, bf16 with beta.  Each tile, last rows and columns missing, one tile to a workgroup and several.  Every element:
int32 bit for bit with exact sums, bf16 with the bound of its sums."""
import pytest
import torch

from gpu_util import check_bf16_product, check_equal, product_i64
from paper_2505_18574_amd import ops
from test_gpu_interleaved import bias_of, matrix, operands, output

pytestmark = pytest.mark.gpu

# the tile that int32 outputs take (choose_tile), the 256 x 256 one on the ping-pong loop: one to a workgroup and several
SHAPES = {"64": (1317, 428, 4560), "128": (1500, 1532, 400), "256x128": (4001, 1596, 272), "256": (3601, 4076, 592), "256, several": (5393, 5388, 336)}


@pytest.mark.parametrize("dword", [False, True])
@pytest.mark.parametrize("kind", ["none", "row", "matrix"])
@pytest.mark.parametrize("tile", SHAPES)
def test_i32(tile, kind, dword):
    M, N, K = SHAPES[tile]
    N = N if dword else N + 4 & ~15
    A, B, Am, Bm = operands(M, N, K - 4 * dword, torch.int8, M + K, dword=dword)
    b = bias_of(kind, M, N, K)
    C = output(M, N, torch.int32, 9)
    ops.ac_gemm_i8_acc32(A, B, b, C[:M])
    check_equal(C[:M], product_i64(Am, Bm) + (0 if b is None else b))
    assert (C[M] == 9).all()


@pytest.mark.parametrize("dword", [False, True])
@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (0.5, -2.0)])
@pytest.mark.parametrize("tile", SHAPES)
def test_bf16(tile, alpha, beta, dword):
    M, N, K = SHAPES[tile]
    N = N if dword else N + 4 & ~7
    K = K // 2 - 2 * dword
    A, B, Am, Bm = operands(M, N, K, torch.bfloat16, M + K, dword=dword)
    old = matrix(M + 1, N, torch.bfloat16, 6).float()
    C = old.clone()
    ops.ac_gemm_bf16(A, B, C[:M], alpha, beta)
    check_bf16_product(Am, Bm, C[:M], alpha, beta, old[:M])
    assert torch.equal(C[M], old[M])
