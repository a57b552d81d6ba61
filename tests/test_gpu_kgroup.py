"""GPU parity of the kernels whose waves share an output tile and take its K tiles in turn (few tiles, any K): edges of the
32 x 32 tile and of the 64- and 128-byte K tiles, waves without a K tile, rings that are never full, a partial last K tile
on every wave, each operand form, both sides of the rules' borders in K and in the tile count.  int8 bit for bit; bf16
against float64 within 4 (K + 2) 2^-24 sum |a b| per element (fp32 sums of exact products in any order)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_bf16_product_in_full, dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu
FORMS = ["plain", "ta", "tb", "tab", "i32"]


def odd(a):
    """The same matrix one element off an aligned address, with an odd pitch."""
    src = dev(a)
    big = torch.zeros((a.shape[0], a.shape[1] + 5), dtype=src.dtype, device="cuda")
    v = big[:, 1:1 + a.shape[1]]
    v.copy_(src)
    return v


def check_i8(form, M, N, K, put=dev, shift=9, act=1, bias_matrix=False):
    A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=M + 2 * N + 3 * K, bias_matrix=bias_matrix)
    ta, tb = form in ("ta", "tab"), form in ("tb", "tab")
    At, Bt = put(np.ascontiguousarray(A.T) if ta else A), put(np.ascontiguousarray(B.T) if tb else B)
    if form == "i32":
        C = put(np.full((M, N), 7, np.int32))
        ops.ac_gemm_i8_acc32(At, Bt, dev(bias), C)
        want = A.astype(np.int64) @ B.astype(np.int64) + bias
    else:
        C = put(np.full((M, N), 7, np.int8))
        if ta or tb:
            ops.ac_gemm_i8_t(At, Bt, dev(bias), C, shift, act, trans_a=ta, trans_b=tb)
        else:
            ops.ac_gemm_i8(At, Bt, dev(bias), C, shift, act)
        want = oracle.gemm_i8(A, B, bias, shift, act)
    np.testing.assert_array_equal(host(C), want)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("M,N,K", [
    (16, 16, 16), (48, 80, 48), (32, 32, 64), (16, 48, 208),   # one K tile or less for every wave
    (64, 32, 512), (80, 16, 528),                              # four waves, then eight
    (48, 48, 1040), (32, 16, 1600), (16, 64, 3264),            # K tiles per wave: two and three, and a partial one
    (32, 48, 4848), (32, 48, 4864), (16, 32, 5008),            # 64- and 128-byte K tiles
    (512, 512, 576), (528, 512, 576), (544, 512, 640), (544, 512, 656),  # 256 and 272 tiles
    (528, 512, 352), (528, 512, 368), (528, 512, 608), (528, 512, 624), (57, 64, 64), (128, 128, 64), (160, 128, 64)])
def test_aligned(form, M, N, K):
    check_i8(form, M, N, K)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("M,N,K", [
    (17, 17, 63), (17, 16, 64), (33, 31, 65), (16, 19, 127), (31, 33, 128), (40, 21, 129), (1, 16, 700), (19, 37, 1023),
    (32, 32, 1025), (35, 18, 2049), (23, 45, 3501), (509, 511, 300), (515, 515, 300), (640, 703, 200), (15, 40, 300), (40, 15, 300)])
def test_any_alignment(form, M, N, K):
    check_i8(form, M, N, K)
    check_i8(form, M, N, K, put=odd, bias_matrix=True)


@pytest.mark.parametrize("shift,act", [(0, 0), (1, 0), (17, 1), (18, 0), (23, 1), (24, 0), (31, 1)])
def test_output_stage(shift, act):
    for put, K in ((dev, 1040), (odd, 1037)):
        check_i8("plain", 40, 48, K, put, shift, act)
        check_i8("plain", 40, 48, K, put, shift, act, bias_matrix=True)


@pytest.mark.parametrize("K", [2592, 2608, 3168, 3184, 3488, 3504, 4096, 4112, 4480, 4496, 7168, 7184])
def test_beside_a_workspace(K):
    """Products that the other kernels would cut over workgroups: both sides of the rule, same bytes."""
    for M, N in ((40, 512), (70, 48), (17, 48), (35, 51), (40, 515)):
        A, B, bias = inputs.gemm_i8_inputs(M, N, K, seed=K + M)
        ws = torch.empty(max(16, ops.ac_gemm_i8_workspace_bytes(M, N, K)), dtype=torch.uint8, device="cuda")
        C = torch.full((M, N), 3, dtype=torch.int8, device="cuda")
        ops.ac_gemm_i8(dev(A), dev(B), dev(bias), C, 13, 0, workspace=ws)
        np.testing.assert_array_equal(host(C), oracle.gemm_i8(A, B, bias, 13, 0))


@pytest.mark.parametrize("M,N,K", [(16, 8, 8), (40, 24, 72), (33, 56, 256), (64, 40, 264), (17, 16, 1000), (48, 8, 2440), (300, 328, 520),
                                   (17, 9, 33), (33, 31, 511), (40, 70, 777), (511, 500, 150), (600, 520, 99)])
@pytest.mark.parametrize("put", [dev, odd])
def test_bf16(M, N, K, put):
    A, B = inputs.gemm_bf16_inputs(M, N, K, seed=M + N + K)
    C = put(np.full((M, N), np.nan, np.float32))
    ops.ac_gemm_bf16(put(A), put(B), C)
    check_bf16_product_in_full(A, B, host(C))
    C0 = np.arange(M * N, dtype=np.float32).reshape(M, N) % 17  # alpha and beta; the sum of C is exact to 2^-24 of its terms
    C = put(C0)
    ops.ac_gemm_bf16(put(A), put(B), C, 0.5, 2.0)
    want = oracle.gemm_bf16(A, B, 0.5, 2.0, C0)
    mag = 0.5 * (np.abs(inputs.bf16_bits_to_f32(A).astype(np.float64)) @ np.abs(inputs.bf16_bits_to_f32(B).astype(np.float64))) + 2 * np.abs(C0)
    assert (np.abs(host(C) - want) <= 4 * (K + 2) * 2.0 ** -24 * mag + 1e-30).all()


@pytest.mark.parametrize("Nb,H,W,Cin,Cout,KH,KW,stride,pad", [
    (1, 9, 7, 16, 16, 3, 3, 1, 1), (2, 14, 13, 48, 80, 5, 5, 1, 2), (3, 15, 15, 336, 48, 3, 3, 2, 1), (1, 6, 5, 1040, 32, 1, 1, 2, 0),
    (2, 9, 9, 48, 16, 7, 7, 1, 3), (1, 40, 33, 32, 16, 1, 32, 1, 16), (9, 30, 31, 32, 48, 3, 3, 1, 1), (1, 5, 5, 16, 16, 2, 2, 3, 0),
    (1, 13, 13, 59, 57, 5, 5, 1, 2), (2, 9, 11, 25, 3, 3, 3, 1, 1), (1, 20, 19, 33, 47, 3, 3, 2, 1), (1, 8, 8, 22, 17, 3, 3, 1, 9),
    (3, 7, 60, 7, 40, 6, 5, 1, 2), (30, 17, 18, 60, 58, 5, 5, 1, 2), (1, 1, 400, 210, 20, 1, 1, 2, 0), (1, 60, 9, 23, 18, 40, 1, 1, 3)])
def test_convolutions(Nb, H, W, Cin, Cout, KH, KW, stride, pad):
    x, w, b = inputs.conv_i8_inputs(Nb, H, W, Cin, Cout, KH, KW, seed=H * W + Cin)
    want = oracle.conv2d_i8(x, w, b, stride, pad, 10, 1)
    out = torch.full(want.shape, 17, dtype=torch.int8, device="cuda")
    ops.ac_conv2d_i8(dev(x), dev(w), dev(b), out, stride, pad, 10, 1)
    np.testing.assert_array_equal(host(out), want)


@pytest.mark.parametrize("M,N,K", [(8193, 32, 624), (16384, 16, 1408), (16383, 32, 1424), (288, 928, 960), (511, 1008, 944), (511, 1008, 976), (300, 932, 956), (4099, 60, 1404)])
def test_int32_on_two_rounds(M, N, K):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + N + K)
    for bias in (b, None):
        C = torch.full((M, N), 9, dtype=torch.int32, device="cuda")
        ops.ac_gemm_i8_acc32(dev(A), dev(B), None if bias is None else dev(bias), C)
        np.testing.assert_array_equal(host(C), (A.astype(np.float64) @ B.astype(np.float64) + (0 if bias is None else bias)).astype(np.int32))  # sums below 2^53


# images, edge, input and output channels, kernel edge, stride: both sides of each line, and the most tiles of two rounds
@pytest.mark.parametrize("Nb,edge,Cin,Cout,k,stride", [
    (1, 40, 384, 16, 5, 1), (2, 9, 400, 16, 5, 1), (2, 9, 432, 16, 5, 1), (1, 14, 352, 32, 5, 1), (1, 14, 384, 32, 5, 1), (1, 20, 128, 48, 7, 1), (1, 20, 160, 64, 7, 1),
    (3, 19, 208, 80, 5, 2), (3, 19, 176, 80, 5, 2), (3, 19, 176, 128, 5, 2), (1, 7, 208, 144, 5, 1), (15, 33, 304, 32, 5, 1), (4, 37, 320, 48, 5, 1), (4, 37, 336, 48, 5, 1),
    (7, 14, 160, 240, 5, 1), (7, 14, 176, 240, 5, 1), (33, 9, 256, 160, 3, 1), (33, 9, 272, 160, 3, 1),
    (3, 31, 192, 128, 5, 1), (3, 31, 208, 128, 5, 1), (13, 16, 208, 112, 5, 1), (13, 16, 224, 112, 5, 1), (17, 15, 256, 96, 5, 1), (17, 15, 272, 96, 5, 1),
    (5, 28, 96, 128, 5, 1), (5, 28, 112, 128, 5, 1), (14, 7, 400, 400, 3, 1), (14, 7, 400, 416, 3, 1)])
def test_convolutions_beside_a_workspace(Nb, edge, Cin, Cout, k, stride):
    x, w, b = inputs.conv_i8_inputs(Nb, edge, edge, Cin, Cout, k, k, seed=edge + Cin + Cout)
    want = oracle.conv2d_i8(x, w, b, stride, k // 2, 11, 1)
    ws = torch.empty(max(16, ops.ac_gemm_i8_workspace_bytes(want.size // Cout, Cout, k * k * Cin)), dtype=torch.uint8, device="cuda")
    for workspace in (ws, None):
        out = torch.full(want.shape, 17, dtype=torch.int8, device="cuda")
        ops.ac_conv2d_i8(dev(x), dev(w), dev(b), out, stride, k // 2, 11, 1, workspace=workspace)
        np.testing.assert_array_equal(host(out), want)


def test_same_bits_on_every_run():
    """The waves' sums are added in one order (with no workspace, the kernels that cut K add them as they come)."""
    A, B = inputs.gemm_bf16_inputs(64, 96, 2400, seed=5)
    outs = []
    for _ in range(5):
        C = torch.empty((64, 96), dtype=torch.float32, device="cuda")
        ops.ac_gemm_bf16(dev(A), dev(B), C)
        outs.append(host(C))
    assert all(np.array_equal(o, outs[0]) for o in outs)
