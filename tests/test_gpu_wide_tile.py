"""Products and convolutions on one round of 64 x 128 tiles (128 x 64 with both operands transposed): every form that takes it, last
rows and columns of a tile that are missing, fewer K tiles than stages, a partial last one, exactly as many tiles as compute
units, bias rows, matrices and none.  The first test, on the host, holds the shapes to the rule."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_bf16_product_in_full, dev, host
from paper_2505_18574_amd import inputs, ops

gpu = pytest.mark.gpu
PRODUCTS = [(2113, 528, 256), (8161, 160, 304), (2049, 816, 640), (300, 3344, 1168), (4200, 272, 4112)]
DWORD_PRODUCTS = [(2113, 532, 320), (1000, 1500, 324), (8161, 132, 1004), (2049, 812, 388)]
BF16 = [(2113, 528, 320), (8161, 160, 328), (2049, 816, 1000)]
DWORD_BF16 = [(2113, 532, 352), (1500, 1000, 502), (8161, 132, 388)]
TRANSPOSED = [("ta", 2128, 528, 272), ("ta", 8160, 160, 1168), ("tb", 2113, 528, 640), ("tb", 8161, 160, 1040), ("tab", 528, 2128, 272), ("tab", 160, 8161 // 16 * 16, 1168),
              ("ta", 2116, 532, 324), ("ta", 1004, 1500, 1004), ("tab", 532, 2116, 256), ("tab", 2052, 812, 1004)]
# images, edge, input and output channels, kernel edge, stride
CONVOLUTIONS = [(8, 29, 80, 176, 3, 1), (51, 24, 544, 192, 1, 2), (110, 19, 576, 128, 1, 2), (3, 83, 64, 352, 3, 2), (9, 22, 128, 384, 2, 1), (23, 27, 128, 256, 2, 2), (1, 90, 32, 144, 3, 1), (16, 41, 96, 208, 3, 2), (60, 25, 336, 80, 1, 2), (5, 75, 112, 192, 5, 2), (12, 32, 240, 80, 5, 1)]

SHIM = """
#include "gemm_rules.hpp"
extern "C" int product(int M, int N, int K, int eb, int dw, int splits) { return ac::wide_product_rule(M, N, (int64_t)K * eb, eb, dw != 0, splits); }
extern "C" int trans(int M, int N, int K, int ta, int tb, int dw) { return ac::wide_trans_rule(M, N, K, ta != 0, tb != 0, dw != 0); }
extern "C" int conv(int M, int N, int K, int taps, int stride, int bytes) { return ac::wide_conv_rule(M, N, K, taps, stride, bytes); }
"""


def conv_sizes(nb, edge, cin, cout, k, stride):
    out = (edge + 2 * (k // 2) - k) // stride + 1
    return nb * out * out, cout, k * k * cin


def test_rule(tmp_path):
    (tmp_path / "shim.cpp").write_text(SHIM)
    so = str(tmp_path / "shim.so")
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_18574_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", csrc, "-o", so, str(tmp_path / "shim.cpp")], check=True)
    rules = ctypes.CDLL(so)
    for M, N, K in PRODUCTS:
        assert rules.product(M, N, K, 1, 0, 1), (M, N, K)
    for M, N, K in DWORD_PRODUCTS:
        assert rules.product(M, N, K, 1, 1, 1), (M, N, K)
    for M, N, K in BF16:
        assert rules.product(M, N, K, 2, 0, 1) and not rules.product(M, N, K, 2, 0, 4), (M, N, K)
    for M, N, K in DWORD_BF16:
        assert rules.product(M, N, K, 2, 1, 1), (M, N, K)
    for form, M, N, K in TRANSPOSED:
        dw = N % 16 != 0 or K % 16 != 0 or ("a" in form and M % 16 != 0)
        assert rules.trans(M, N, K, "a" in form, "b" in form, dw), (form, M, N, K)
    for c in CONVOLUTIONS:
        M, N, K = conv_sizes(*c)
        assert rules.conv(M, N, K, c[4] ** 2, c[5], c[0] * c[1] ** 2 * c[2] + K * N), c
    # a round of 64 x 64 tiles, two rounds of these, K too short, slices that are ahead, columns that are whole lines anyway
    assert rules.product(16384, 128, 512, 1, 0, 1)  # 256 tiles: one to each unit
    assert not rules.product(16385, 128, 512, 1, 0, 1) and not rules.product(1024, 1024, 1024, 1, 0, 1)
    assert not rules.product(2113, 528, 240, 1, 0, 1) and not rules.product(936, 1200, 7808, 1, 0, 2) and rules.product(936, 1200, 7808, 1, 0, 1)
    # tiles of one wave: few of 64 bytes of K whose windows overlap; their other K, more tiles, no overlap, and K that is not theirs
    for M, N, K, taps, stride, takes in [(6348, 160, 576, 9, 1, 0), (6156, 144, 576, 9, 2, 0), (5832, 176, 320, 4, 1, 0), (5887, 176, 448, 4, 1, 0), (4851, 288, 576, 9, 1, 0), (7803, 192, 576, 9, 1, 0), (3200, 416, 576, 9, 2, 1), (4050, 368, 576, 9, 1, 1),
                                         (5239, 352, 576, 9, 2, 1), (4225, 384, 512, 4, 1, 1), (13068, 112, 576, 1, 2, 1), (7344, 192, 544, 1, 2, 1), (5480, 208, 608, 1, 2, 1), (5832, 208, 640, 4, 1, 1)]:
        assert rules.conv(M, N, K, taps, stride, 5000000) == takes, (M, N, K, taps, stride)
    assert not rules.trans(2113, 532, 1004, 0, 1, 1) and not rules.conv(11264, 128, 3136, 49, 1, 1 << 20)


def int8_case(form, M, N, K, bias):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + 2 * N + 3 * K, bias_matrix=bias == "matrix")
    if bias == "none":
        b = np.zeros_like(b)
    return A, B, b, None if bias == "none" else dev(b)


@gpu
@pytest.mark.parametrize("bias", ["row", "none", "matrix"])
@pytest.mark.parametrize("M,N,K", PRODUCTS + DWORD_PRODUCTS)
def test_int8(M, N, K, bias):
    A, B, b, t = int8_case("plain", M, N, K, bias)
    C = torch.full((M, N), 9, dtype=torch.int8, device="cuda")
    nb = ops.ac_gemm_i8_workspace_bytes(M, N, K)
    ops.ac_gemm_i8(dev(A), dev(B), t, C, 9, 1, workspace=torch.empty(nb, dtype=torch.uint8, device="cuda") if nb else None)
    np.testing.assert_array_equal(host(C), oracle.gemm_i8(A, B, b, 9, 1))
    C32 = torch.full((M, N), 9, dtype=torch.int32, device="cuda")
    ops.ac_gemm_i8_acc32(dev(A), dev(B), t, C32)
    np.testing.assert_array_equal(host(C32), (A.astype(np.float64) @ B.astype(np.float64) + b).astype(np.int32))  # sums below 2^53


@gpu
@pytest.mark.parametrize("form,M,N,K", TRANSPOSED)
def test_transposed(form, M, N, K):
    A, B, b, t = int8_case(form, M, N, K, "row")
    ta, tb = "a" in form, "b" in form
    C = torch.full((M, N), 9, dtype=torch.int8, device="cuda")
    ops.ac_gemm_i8_t(dev(A.T) if ta else dev(A), dev(B.T) if tb else dev(B), t, C, 9, 0, trans_a=ta, trans_b=tb)
    np.testing.assert_array_equal(host(C), oracle.gemm_i8(A, B, b, 9, 0))


@gpu
@pytest.mark.parametrize("M,N,K", BF16 + DWORD_BF16)
def test_bf16(M, N, K):
    A, B = inputs.gemm_bf16_inputs(M, N, K, seed=M + N + K)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    ops.ac_gemm_bf16(dev(A), dev(B), C)
    check_bf16_product_in_full(A, B, host(C))


@gpu
@pytest.mark.parametrize("nb,edge,cin,cout,k,stride", CONVOLUTIONS)
def test_convolutions(nb, edge, cin, cout, k, stride):
    x, w, b = inputs.conv_i8_inputs(nb, edge, edge, cin, cout, k, k, seed=edge + cin + cout)
    M, N, K = conv_sizes(nb, edge, cin, cout, k, stride)
    want = oracle.conv2d_i8(x, w, b, stride, k // 2, 9, 1)
    out = torch.full(want.shape, 9, dtype=torch.int8, device="cuda")
    ops.ac_conv2d_i8(dev(x), dev(w), dev(b), out, stride, k // 2, 9, 1)
    np.testing.assert_array_equal(host(out), want)
