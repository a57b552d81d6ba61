"""GPU parity of the direct-to-LDS products on operands aligned to 4 bytes and no more: every operand form, K and extents that
end inside a 16-byte chunk, a last K tile of one dword up to a whole one, one K tile and none before it, tiles of 32 to 256 rows
and columns, K slices, views off an aligned address; what lies behind a row's end must not count."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_bf16_product_in_full, dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu


def view(a, shift, fill):
    """A matrix `shift` elements into rows that are 2 * shift longer, surrounded by `fill`."""
    src = dev(a)
    big = torch.full((a.shape[0], a.shape[1] + 2 * shift), fill, dtype=torch.float32, device="cuda").to(src.dtype)
    v = big[:, shift:shift + a.shape[1]]
    v.copy_(src)
    return v


def check_i8(form, M, N, K, shift=0, workspace=False):
    A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=M + 2 * N + 3 * K)
    ta, tb = form in ("ta", "tab"), form in ("tb", "tab")
    put = (lambda x: view(x, shift, 77)) if shift else dev
    At, Bt = put(np.ascontiguousarray(A.T) if ta else A), put(np.ascontiguousarray(B.T) if tb else B)
    if form == "i32":
        C = torch.full((M, N), 7, dtype=torch.int32, device="cuda")
        ops.ac_gemm_i8_acc32(At, Bt, dev(bias), C)
        want = (A.astype(np.int64) @ B.astype(np.int64) + bias).astype(np.int32) if M * N * K < 1 << 27 else A.astype(np.float64) @ B.astype(np.float64) + bias
    else:
        C = view(np.full((M, N), 7, np.int8), 4, 9) if shift else torch.full((M, N), 7, dtype=torch.int8, device="cuda")
        if ta or tb:
            ops.ac_gemm_i8_t(At, Bt, dev(bias), C, 9, 1, trans_a=ta, trans_b=tb)
        else:
            nb = ops.ac_gemm_i8_workspace_bytes(M, N, K) if workspace else 0
            ops.ac_gemm_i8(At, Bt, dev(bias), C, 9, 1, workspace=torch.empty(nb, dtype=torch.uint8, device="cuda") if nb else None)
        want = oracle.gemm_i8(A, B, bias, 9, 1)
    np.testing.assert_array_equal(host(C), want)


@pytest.mark.parametrize("form", ["plain", "ta", "tb", "tab", "i32"])
@pytest.mark.parametrize("M,N,K", [
    (16, 16, 20), (20, 20, 16), (36, 52, 60), (20, 16, 64), (28, 36, 68), (32, 32, 124), (60, 20, 128), (36, 100, 132), (40, 20, 516),
    (20, 44, 1004), (48, 16, 2052),                                        # waves in turn
    (1004, 1004, 252), (1000, 1000, 128), (1300, 1292, 388), (516, 3004, 1028)])  # 64- and 128-wide tiles
def test_forms(form, M, N, K):
    check_i8(form, M, N, K)
    check_i8(form, M, N, K, shift=4)


# what the product's plan and the rule for these operands choose: test_gemm_rules.py holds each shape to its tile (transposed
# operands take 128 for 192)
DIRECT_TILES = {64: [(556, 8284, 128), (524, 8372, 152)], 128: [(788, 8432, 140), (5448, 328, 2088)], 192: [(708, 8900, 136), (708, 8908, 388)],
                256: [(916, 8908, 132), (796, 9500, 292)]}


@pytest.mark.parametrize("form", ["plain", "ta", "tb", "tab"])
@pytest.mark.parametrize("M,N,K", [shape for shapes in DIRECT_TILES.values() for shape in shapes])
def test_direct_tiles(form, M, N, K):
    check_i8(form, M, N, K, shift=4)


@pytest.mark.parametrize("form", ["plain", "tab", "i32"])
@pytest.mark.parametrize("M,N,K", [(4100, 4108, 60), (4100, 4108, 256), (3076, 3588, 324), (12292, 1028, 260)])
def test_wide_tiles(form, M, N, K):
    check_i8(form, M, N, K)


@pytest.mark.parametrize("M,N,K", [(52, 516, 4612), (132, 100, 9004), (20, 2052, 8196)])
def test_slices(M, N, K):
    check_i8("plain", M, N, K, workspace=True)


@pytest.mark.parametrize("M,N,K", [(17, 20, 18), (33, 36, 66), (40, 52, 126), (64, 20, 130), (35, 44, 514), (1000, 1004, 202), (1300, 1292, 322), (4099, 4108, 34), (2051, 2572, 130)])
@pytest.mark.parametrize("shift", [0, 4])
def test_bf16(M, N, K, shift):
    """The rows' surroundings are NaN: what is read of them must not reach a sum."""
    A, B = inputs.gemm_bf16_inputs(M, N, K, seed=M + N + K)
    At, Bt = (view(A, shift, float("nan")), view(B, shift, float("nan"))) if shift else (dev(A), dev(B))
    C = torch.full((M, N), float("nan"), device="cuda")
    ops.ac_gemm_bf16(At, Bt, C)
    check_bf16_product_in_full(A, B, host(C))


def test_bf16_neighbouring_rows_of_infinities():
    A, B = inputs.gemm_bf16_inputs(40, 36, 70, seed=4)
    At, Bt = dev(A), dev(B)
    At[7] = float("inf")
    At[9] = float("nan")
    C = torch.empty((40, 36), device="cuda")
    ops.ac_gemm_bf16(At, Bt, C)
    keep = [r for r in range(40) if r not in (7, 9)]
    check_bf16_product_in_full(A[keep], B, host(C)[keep])
    assert not np.isfinite(host(C)[[7, 9]]).any()


def test_bf16_deep_k_is_the_same_with_and_without_a_workspace():
    A, B = inputs.gemm_bf16_inputs(36, 68, 7002, seed=6)
    ws = torch.empty(max(16, ops.ac_gemm_bf16_workspace_bytes(36, 68, 7002)), dtype=torch.uint8, device="cuda")
    outs = []
    for w in (ws, None, ws, None):
        C = torch.full((36, 68), float("nan"), device="cuda")
        ops.ac_gemm_bf16_ws(dev(A), dev(B), C, workspace=w)
        outs.append(host(C))
    check_bf16_product_in_full(A, B, outs[0])
    assert all(np.array_equal(o, outs[0]) for o in outs)
