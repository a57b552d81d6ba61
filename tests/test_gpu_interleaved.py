"""GPU parity of the interleaved K loop of the 256 x 256 tiles: every count of last trips (K tiles of 64 bytes modulo the four
stages), a partial last K tile, last rows and columns that are missing, shifts at both ends of its output stage's range, several
tiles to a workgroup with the next one's prefetch, each operand form it has.  int8 bit for bit, bf16 against the bound of fp32
sums.  test_gemm_rules.py holds each shape to the loop."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_bf16_product_in_full, dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu

# 184 to 256 tiles of 256 x 256, one round of them
NAMED_I8 = [(3600, 3344, 2048), (3585, 3600, 2064), (4096, 4096, 1024), (3839, 3984, 1104), (3910, 4096, 1152), (3600, 3344, 2240 + 48)]
NAMED_BF16 = [(3600, 3600, 512), (3585, 3856, 520), (4096, 4096, 544), (3839, 3984, 576), (3910, 3600, 608), (3600, 3344, 1032)]
# (M, N, K, out, trans_a, trans_b): more tiles of 256 x 256 than compute units; K whole 16 bytes and whole dwords
CHOSEN = [(8200, 4112, 2112, "i8", False, False), (8200, 4112, 1040, "i8", False, True), (8208, 8208, 592, "i8", True, True), (4100, 4112, 2064, "i32", False, False),
          (8200, 4100, 2116, "i8", False, False), (8200, 4100, 1092, "i8", False, True), (4100, 4100, 2084, "i32", False, False)]
CHOSEN_BF16 = [(8200, 8208, 520), (8200, 8204, 518)]


# the 128 x 256 tiles that a product without a plan takes: on one round of them and on more
CHOSEN_128X256 = [(1105, 4544, 2064), (1361, 4736, 2176), (2257, 3232, 3136), (3297, 6960, 1296), (6049, 3008, 2240)]


# ... and A^T B^T products
CHOSEN_AT_BT = [(1712, 3584, 512), (2128, 2192, 592), (1040, 4112, 1136), (4464, 1744, 704)]


@pytest.mark.parametrize("shift,kind", [(1, "row"), (17, "row"), (9, "none"), (9, "matrix"), (18, "row"), (0, "row")])
@pytest.mark.parametrize("M,N,K", NAMED_I8)
def test_named_tile_i8(M, N, K, shift, kind):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + N + K + shift, bias_matrix=kind == "matrix")
    t = None if kind == "none" else dev(b)
    r = rows_of(M)
    acc = (A[r].astype(np.float64) @ B.astype(np.float64)).astype(np.int64) + (0 if t is None else b[r] if kind == "matrix" else b)
    for act in (0, 1):
        C = torch.full((M + 1, N), 9, dtype=torch.int8, device="cuda")
        ops.ac_gemm_i8_planned(dev(A), dev(B), t, C[:M], shift, act, 256, 1)
        np.testing.assert_array_equal(host(C)[r], oracle.requantise_vec(acc, shift, act))
        assert (host(C[M]) == 9).all()  # nothing behind the last row


@pytest.mark.parametrize("M,N,K", NAMED_BF16)
def test_named_tile_bf16(M, N, K):
    A, B = inputs.gemm_bf16_inputs(M, N, K, seed=M + N + K)
    C = torch.full((M + 1, N), float("nan"), dtype=torch.float32, device="cuda")
    ops.ac_gemm_bf16_planned(dev(A), dev(B), C[:M], 1.0, 0.0, 256, 1)
    r = rows_of(M)
    check_bf16_product_in_full(A[r], B, host(C)[r])
    assert np.isnan(host(C[M])).all()
    old = np.random.default_rng(M).standard_normal((M, N)).astype(np.float32)
    C = dev(old)
    ops.ac_gemm_bf16_planned(dev(A), dev(B), C, 0.5, -2.0, 256, 1)
    want = oracle.gemm_bf16(A[r], B, 0.5, -2.0, old[r])
    assert np.linalg.norm(host(C)[r] - want) <= 1e-3 * np.linalg.norm(want)


def rows_of(M):
    """Rows at the edges of MFMA tiles, wave tiles and workgroup tiles, and the last ones."""
    return sorted({r for e in range(0, M, 256) for r in (e, e + 15, e + 16, e + 127, e + 128, e + 255) if r < M} | {M - 2, M - 1})


@pytest.mark.parametrize("M,N,K,out,ta,tb", CHOSEN)
def test_several_tiles_to_a_workgroup_i8(M, N, K, out, ta, tb):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + N + K)
    At, Bt = dev(A.T if ta else A), dev(B.T if tb else B)
    C = torch.full((M, N), 9, dtype=torch.int32 if out == "i32" else torch.int8, device="cuda")
    if out == "i32":
        ops.ac_gemm_i8_acc32(At, Bt, dev(b), C)
    elif ta or tb:
        ops.ac_gemm_i8_t(At, Bt, dev(b), C, 11, 0, trans_a=ta, trans_b=tb)
    else:
        ops.ac_gemm_i8(At, Bt, dev(b), C, 11, 0)
    r = rows_of(M)
    acc = (A[r].astype(np.float64) @ B.astype(np.float64)).astype(np.int64) + b  # exact: below 2^53
    np.testing.assert_array_equal(host(C)[r], acc if out == "i32" else oracle.requantise_vec(acc, 11, 0))


@pytest.mark.parametrize("shift,kind", [(1, "row"), (17, "none"), (11, "matrix"), (18, "row")])
@pytest.mark.parametrize("M,N,K", CHOSEN_128X256)
def test_128x256(M, N, K, shift, kind):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + N + K, bias_matrix=kind == "matrix")
    t = None if kind == "none" else dev(b)
    C = torch.full((M + 1, N), 9, dtype=torch.int8, device="cuda")
    ops.ac_gemm_i8(dev(A), dev(B), t, C[:M], shift, 1)
    r = rows_of(M)
    acc = (A[r].astype(np.float64) @ B.astype(np.float64)).astype(np.int64) + (0 if t is None else b[r] if kind == "matrix" else b)
    np.testing.assert_array_equal(host(C)[r], oracle.requantise_vec(acc, shift, 1))
    assert (host(C[M]) == 9).all()


@pytest.mark.parametrize("shift,kind", [(2, "row"), (17, "none"), (11, "matrix")])
@pytest.mark.parametrize("M,N,K", CHOSEN_AT_BT)
def test_128x256_at_bt(M, N, K, shift, kind):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + N + K, bias_matrix=kind == "matrix")
    t = None if kind == "none" else dev(b)
    C = torch.full((M + 1, N), 9, dtype=torch.int8, device="cuda")
    ops.ac_gemm_i8_t(dev(A.T), dev(B.T), t, C[:M], shift, 1, trans_a=True, trans_b=True)
    r = rows_of(M)
    acc = (A[r].astype(np.float64) @ B.astype(np.float64)).astype(np.int64) + (0 if t is None else b[r] if kind == "matrix" else b)
    np.testing.assert_array_equal(host(C)[r], oracle.requantise_vec(acc, shift, 1))
    assert (host(C[M]) == 9).all()


@pytest.mark.parametrize("M,N,K", CHOSEN_BF16)
def test_several_tiles_to_a_workgroup_bf16(M, N, K):
    A, B = inputs.gemm_bf16_inputs(M, N, K, seed=M + N + K)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    ops.ac_gemm_bf16(dev(A), dev(B), C)
    r = rows_of(M)
    check_bf16_product_in_full(A[r], B, host(C)[r])


def test_output_beside_other_columns():
    """C with a pitch of its own: the columns behind N stay."""
    M, N, K = NAMED_I8[1]
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=5)
    C = torch.full((M, N + 16), 9, dtype=torch.int8, device="cuda")
    ops.ac_gemm_i8_planned(dev(A), dev(B), dev(b), C[:, :N], 9, 1, 256, 1)
    r = rows_of(M)
    acc = (A[r].astype(np.float64) @ B.astype(np.float64)).astype(np.int64) + b
    np.testing.assert_array_equal(host(C)[r][:, :N], oracle.requantise_vec(acc, 9, 1))
    assert (host(C)[:, N:] == 9).all()
