"""GPU parity of the kernel for operands of any size, pitch and alignment, at the sizes where its loads change form:
chunk, tile and pipeline edges of every dimension, rows and whole operands shorter than a 16-byte chunk, views at odd
addresses, windows that hang over every edge of an image.  int8 bit for bit; bf16 within 4 (K + 2) 2^-24 of the sum of
magnitudes per element (exact products, K fp32 additions)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu

# (M, N, K): one under / over a chunk, a tile of 64 and of 128, whole K tiles (128 bytes), 3 and 5 tiles in flight
SIZES = [(1, 1, 1), (3, 2, 1), (1, 5, 3), (2, 7, 15), (5, 16, 17), (63, 15, 127), (65, 17, 128), (64, 65, 129), (33, 63, 383),
         (31, 129, 385), (7, 127, 641), (129, 33, 769), (200, 50, 1000), (1, 300, 77), (300, 1, 1111), (1441, 1003, 97)]


def odd_view(a):
    """The array in device memory one element off an aligned address, rows an odd pitch apart."""
    buf = torch.zeros((a.shape[0], a.shape[1] + 3), dtype=dev(a).dtype, device="cuda")
    view = buf[:, 1:1 + a.shape[1]]
    view.copy_(dev(a))
    return view


@pytest.mark.parametrize("M,N,K", SIZES)
def test_int8_every_layout(M, N, K):
    A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=M + 3 * N + 7 * K)
    want = oracle.gemm_i8(A, B, bias, 9, 0)
    At, Bt = np.zeros((K, M), np.int8) + A.T, np.zeros((N, K), np.int8) + B.T
    for put in (dev, odd_view):
        for ta, tb in ((False, False), (True, False), (False, True), (True, True)):
            C = torch.full((M, N), 33, dtype=torch.int8, device="cuda")
            ops.ac_gemm_i8_t(put(At if ta else A), put(Bt if tb else B), dev(bias), C, 9, 0, trans_a=ta, trans_b=tb)
            np.testing.assert_array_equal(host(C), want, err_msg=f"{put.__name__} ta={ta} tb={tb}")
        raw = torch.full((M, N), 33, dtype=torch.int32, device="cuda")
        ops.ac_gemm_i8_acc32(put(A), put(B), dev(bias), raw)
        np.testing.assert_array_equal(host(raw), A.astype(np.int64) @ B.astype(np.int64) + bias)


@pytest.mark.parametrize("M,N,K", SIZES)
def test_bf16(M, N, K):
    A, B = inputs.gemm_bf16_inputs(M, N, K, seed=M + 3 * N + 7 * K)
    want = oracle.gemm_bf16(A, B)
    mag = np.abs(inputs.bf16_bits_to_f32(A).astype(np.float64)) @ np.abs(inputs.bf16_bits_to_f32(B).astype(np.float64))
    for put in (dev, odd_view):
        C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        ops.ac_gemm_bf16(put(A), put(B), C)
        assert (np.abs(host(C) - want) <= 4.0 * (K + 2) * 2.0 ** -24 * mag + 1e-30).all(), put.__name__


def test_bf16_neighbours_of_a_row_stay_out():
    """The bytes that follow a row (of K and of N) in memory are infinities: none may reach a product."""
    M, N, K = 70, 75, 203
    A, B = inputs.gemm_bf16_inputs(M, N, K, seed=5)
    Ai = torch.full((M, K + 9), float("inf"), dtype=torch.bfloat16, device="cuda")
    Bi = torch.full((K + 9, N + 9), float("inf"), dtype=torch.bfloat16, device="cuda")
    Ai[:, 3:3 + K].copy_(dev(A))
    Bi[4:4 + K, 3:3 + N].copy_(dev(B))
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    ops.ac_gemm_bf16(Ai[:, 3:3 + K], Bi[4:4 + K, 3:3 + N], C)
    got, want = host(C), oracle.gemm_bf16(A, B)
    assert np.isfinite(got).all() and np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)


@pytest.mark.parametrize("M,N,K", [(44, 316, 1992), (17, 33, 5001), (49, 1000, 2305)])
def test_int8_cut_along_k(M, N, K):
    A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=K)
    want = oracle.gemm_i8(A, B, bias, 12, 1)
    ws = torch.full((ops.ac_gemm_i8_workspace_bytes(M, N, K),), 0x5A, dtype=torch.uint8, device="cuda")
    assert ws.numel() > 0
    C = torch.full((M, N), 33, dtype=torch.int8, device="cuda")
    ops.ac_gemm_i8(dev(A), dev(B), dev(bias), C, 12, 1, workspace=ws)
    np.testing.assert_array_equal(host(C), want)


@pytest.mark.parametrize("Nb,H,W,Cin,Cout,KH,KW,stride,pad", [
    (2, 37, 41, 3, 64, 7, 7, 2, 3),     # few channels: windows over every edge
    (1, 5, 3, 1, 1, 3, 3, 1, 1),        # an image of 15 bytes
    (1, 4, 4, 1, 17, 3, 3, 1, 1),       # an image of exactly one chunk
    (3, 2, 2, 1, 5, 2, 2, 1, 0),        # a weight array of 20 bytes, rows of 5
    (1, 1, 1, 3, 8, 5, 5, 1, 2),        # everything but one tap is padding
    (2, 9, 9, 4, 16, 4, 4, 1, 0),       # runs of exactly one chunk
    (2, 9, 9, 17, 31, 3, 3, 2, 1),      # runs of three chunks and three bytes
    (1, 20, 20, 16, 32, 7, 7, 1, 3),    # more than 32 taps
    (2, 13, 11, 59, 57, 5, 5, 1, 2),    # a run longer than two K tiles
    (1, 6, 6, 2, 100, 1, 1, 1, 0),      # 1 x 1, a plain product with K = 2
    (4, 40, 40, 5, 130, 3, 3, 1, 1),    # tiles of 128
])
def test_convolutions(Nb, H, W, Cin, Cout, KH, KW, stride, pad):
    x, w, b = inputs.conv_i8_inputs(Nb, H, W, Cin, Cout, KH, KW, seed=H * W + Cin)
    want = oracle.conv2d_i8(x, w, b, stride, pad, 8, 1)
    nbytes = ops.ac_gemm_i8_workspace_bytes(want.shape[0] * want.shape[1] * want.shape[2], Cout, KH * KW * Cin)
    for ws in (None, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None):
        out = torch.full(want.shape, 17, dtype=torch.int8, device="cuda")
        ops.ac_conv2d_i8(dev(x), dev(w), dev(b), out, stride, pad, 8, 1, workspace=ws)
        np.testing.assert_array_equal(host(out), want)


@pytest.mark.parametrize("KH,KW,stride,pad", [(3, 3, 1, 1), (1, 1, 2, 0), (1, 1, 1, 1), (7, 7, 2, 3), (1, 1, 1, 0)])
def test_convolutions_without_input_channels(KH, KW, stride, pad):
    """Empty operands (null addresses): every output is the stage of its bias, with and without a workspace or a plan."""
    Nb, H, W, Cout = 2, 9, 8, 37
    x = torch.empty((Nb, H, W, 0), dtype=torch.int8, device="cuda")
    w = torch.empty((KH, KW, 0, Cout), dtype=torch.int8, device="cuda")
    assert x.data_ptr() == 0 and w.data_ptr() == 0
    b = np.random.default_rng(3).integers(-40000, 40000, Cout).astype(np.int32)
    shape = (Nb, (H + 2 * pad - KH) // stride + 1, (W + 2 * pad - KW) // stride + 1, Cout)
    for bias, sums in ((dev(b), b), (None, np.zeros_like(b))):
        want = np.broadcast_to(oracle.requantise_vec(sums, 8, 0), shape)
        for ws, plan in ((None, None), (torch.empty(4096, dtype=torch.uint8, device="cuda"), None), (None, (64, 1)), (None, (128, 1))):
            out = torch.full(shape, 17, dtype=torch.int8, device="cuda")
            ops.ac_conv2d_i8(x, w, bias, out, stride, pad, 8, 0, workspace=ws, plan=plan)
            np.testing.assert_array_equal(host(out), want, err_msg=f"{ws is not None} {plan}")


@pytest.mark.parametrize("M,N,K", [(9000, 8, 16), (9000, 8, 17), (9000, 9, 16), (8, 9000, 16), (9, 9000, 16), (9000, 14, 15), (15, 9000, 3),
                                   (9000, 15, 16), (16, 16, 16), (15, 16, 16), (1, 1, 16), (1, 70000, 16), (70000, 1, 16)])
def test_short_products(M, N, K):
    """Both sides of the rule that computes products of few terms one output to a thread, every layout and type."""
    A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=M + 3 * N + 7 * K)
    sums = (A.astype(np.float64) @ B.astype(np.float64) + bias).astype(np.int64)
    want = oracle.requantise_vec(sums, 7, 0)
    At, Bt = np.zeros((K, M), np.int8) + A.T, np.zeros((N, K), np.int8) + B.T
    matrix = np.broadcast_to(bias, (M, N)).astype(np.int32)
    for put in (dev, odd_view):
        for ta, tb in ((False, False), (True, False), (False, True), (True, True)):
            C = torch.full((M, N), 33, dtype=torch.int8, device="cuda")
            ops.ac_gemm_i8_t(put(At if ta else A), put(Bt if tb else B), dev(matrix if ta else bias), C, 7, 0, trans_a=ta, trans_b=tb)
            np.testing.assert_array_equal(host(C), want, err_msg=f"{put.__name__} ta={ta} tb={tb}")
        raw = torch.full((M, N), 33, dtype=torch.int32, device="cuda")
        ops.ac_gemm_i8_acc32(put(A), put(B), dev(bias), raw)
        np.testing.assert_array_equal(host(raw), sums)
        A2, B2 = inputs.gemm_bf16_inputs(M, N, K, seed=K)
        a, b = inputs.bf16_bits_to_f32(A2).astype(np.float64), inputs.bf16_bits_to_f32(B2).astype(np.float64)
        C0 = torch.rand((M, N), dtype=torch.float32, device="cuda")
        Cf = C0.clone()
        ops.ac_gemm_bf16(put(A2), put(B2), Cf, alpha=0.5, beta=2.0)
        c0 = host(C0).astype(np.float64)
        assert (np.abs(host(Cf) - (0.5 * (a @ b) + 2 * c0)) <= 4.0 * (K + 2) * 2.0 ** -24 * (np.abs(a) @ np.abs(b) + 2 * c0) + 1e-30).all(), put.__name__


@pytest.mark.parametrize("M,N,K", [(32768, 32, 40), (32769, 32, 200), (32897, 33, 70), (33001, 1, 131), (40000, 15, 700), (32900, 31, 128)])
def test_tall_and_narrow(M, N, K):
    """Both sides of the rule that gives tall outputs of at most 32 columns tiles of 128 x 32, every layout."""
    A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=M + 3 * N + 7 * K)
    sums = (A.astype(np.float64) @ B.astype(np.float64) + bias).astype(np.int64)
    want = oracle.requantise_vec(sums, 9, 1)
    At, Bt = np.zeros((K, M), np.int8) + A.T, np.zeros((N, K), np.int8) + B.T
    for ta, tb in ((False, False), (True, False), (False, True), (True, True)):
        C = torch.full((M, N), 33, dtype=torch.int8, device="cuda")
        ops.ac_gemm_i8_t(odd_view(At if ta else A), odd_view(Bt if tb else B), dev(bias), C, 9, 1, trans_a=ta, trans_b=tb)
        np.testing.assert_array_equal(host(C), want, err_msg=f"ta={ta} tb={tb}")
    raw = torch.full((M, N), 33, dtype=torch.int32, device="cuda")
    ops.ac_gemm_i8_acc32(odd_view(A), odd_view(B), dev(bias), raw)
    np.testing.assert_array_equal(host(raw), sums)
    if K % 2 == 0:
        A2, B2 = inputs.gemm_bf16_inputs(M, N, K // 2, seed=K)
        a, b = inputs.bf16_bits_to_f32(A2).astype(np.float64), inputs.bf16_bits_to_f32(B2).astype(np.float64)
        Cf = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        ops.ac_gemm_bf16(odd_view(A2), odd_view(B2), Cf)
        assert (np.abs(host(Cf) - a @ b) <= 4.0 * (K // 2 + 2) * 2.0 ** -24 * (np.abs(a) @ np.abs(b)) + 1e-30).all()


# K tiles of 128 bytes against the pipeline of the whole tiles: none, 1 .. 2 R + 2 of them (steady trips start at 2 R + 1,
# R = 2), with and without a partial tile; tiles of 64 x 64, 128 x 64 (more than 256 of the former) and 128 x 128
@pytest.mark.parametrize("M,N", [(61, 67), (1030, 1027), (1985, 1410)])
@pytest.mark.parametrize("K", [100, 128, 131, 256, 300, 384, 512, 520, 640, 641, 768, 896, 1000])
def test_pipeline_edges(M, N, K):
    A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=M + 3 * N + 7 * K)
    want = A.astype(np.float64) @ B.astype(np.float64) + bias  # (exact: sums below 2^53)
    C = torch.full((M, N), 33, dtype=torch.int32, device="cuda")
    ops.ac_gemm_i8_acc32(odd_view(A), odd_view(B), dev(bias), C)
    np.testing.assert_array_equal(host(C), want.astype(np.int64))
    q = torch.full((M, N), 33, dtype=torch.int8, device="cuda")
    matrix = np.broadcast_to(bias, (M, N)).astype(np.int32)
    for b in (dev(bias), dev(matrix)):
        ops.ac_gemm_i8(odd_view(A), odd_view(B), b, q, 9, 0)
        np.testing.assert_array_equal(host(q), np.clip(np.rint(want / 512), -128, 127).astype(np.int8))  # halves to even
    if K % 2 == 0:
        A2, B2 = inputs.gemm_bf16_inputs(M, N, K // 2, seed=K)
        a, b = inputs.bf16_bits_to_f32(A2).astype(np.float64), inputs.bf16_bits_to_f32(B2).astype(np.float64)
        Cf = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        ops.ac_gemm_bf16(odd_view(A2), odd_view(B2), Cf)
        assert (np.abs(host(Cf) - a @ b) <= 4.0 * (K // 2 + 2) * 2.0 ** -24 * (np.abs(a) @ np.abs(b)) + 1e-30).all()


@pytest.mark.parametrize("M,N,K", [
    (15, 40, 300), (16, 40, 300), (17, 15, 300), (40, 15, 129), (40, 16, 300), (70, 33, 15), (70, 33, 16), (9, 9, 700),  # one tile and a few
    (210, 1200, 13), (1200, 210, 15), (40000, 9, 100), (33000, 7, 15), (1441, 1003, 15), (15, 66000, 17)])                # each tile shape
def test_rows_of_about_a_chunk(M, N, K):
    """Rows of a K-strided operand, and K itself, on both sides of the 16 bytes from which whole tiles need no guard."""
    A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=M + N + K)
    want = oracle.gemm_i8(A, B, bias, 7, 1)
    At, Bt = np.ascontiguousarray(A.T), np.ascontiguousarray(B.T)
    for put in (dev, odd_view):
        for ta, tb in ((False, False), (True, False), (False, True), (True, True)):
            C = torch.full((M, N), 33, dtype=torch.int8, device="cuda")
            ops.ac_gemm_i8_t(put(At if ta else A), put(Bt if tb else B), dev(bias), C, 7, 1, trans_a=ta, trans_b=tb)
            np.testing.assert_array_equal(host(C), want, err_msg=f"{put.__name__} ta={ta} tb={tb}")
    for K2 in (7, 8, 9):  # bf16: rows of 14, 16 and 18 bytes
        A, B = inputs.gemm_bf16_inputs(min(M, 700), min(N, 700), K2, seed=K2)
        C = torch.full((A.shape[0], B.shape[1]), float("nan"), dtype=torch.float32, device="cuda")
        ops.ac_gemm_bf16(odd_view(A), odd_view(B), C)
        mag = np.abs(inputs.bf16_bits_to_f32(A).astype(np.float64)) @ np.abs(inputs.bf16_bits_to_f32(B).astype(np.float64))
        assert (np.abs(host(C) - oracle.gemm_bf16(A, B)) <= 4.0 * (K2 + 2) * 2.0 ** -24 * mag + 1e-30).all()
