"""Int8 products and convolutions of at most 32 columns on many rows (128 x 32 tiles): a last tile that is one row short or has one row,
fewer K tiles than stages, a partial last one, the sizes at which the rule begins, strides, 1 x 1 kernels with a stride and single
sixteens of channels, bias rows, matrices and none, with a workspace and without."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bias", ["row", "none", "matrix"])
@pytest.mark.parametrize("M,N,K", [(16385, 16, 16), (16512, 32, 128), (16511, 32, 144), (33025, 16, 384), (20001, 32, 400), (131072, 16, 112), (131073, 16, 128), (131073, 16, 112), (40000, 32, 2064), (50000, 32, 2064)])
def test_products(M, N, K, bias):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + 2 * N + 3 * K, bias_matrix=bias == "matrix")
    if bias == "none":
        b = np.zeros_like(b)
    C = torch.full((M, N), 9, dtype=torch.int8, device="cuda")
    ops.ac_gemm_i8(dev(A), dev(B), None if bias == "none" else dev(b), C, 9, 1)
    np.testing.assert_array_equal(host(C), oracle.gemm_i8(A, B, b, 9, 1))


# images, edge, input and output channels, kernel edge, stride
@pytest.mark.parametrize("workspace", [False, True])
@pytest.mark.parametrize("nb,edge,cin,cout,k,stride", [
    (5, 58, 80, 16, 3, 1), (17, 32, 48, 32, 3, 1), (17, 63, 48, 16, 3, 2), (70, 31, 64, 32, 3, 2), (80, 29, 32, 32, 5, 2), (6, 53, 16, 32, 7, 1), (6, 53, 144, 16, 5, 1), (30, 47, 208, 32, 1, 2), (9, 129, 48, 16, 1, 3), (260, 31, 64, 32, 3, 2), (35, 96, 144, 16, 3, 3), (30, 72, 80, 16, 3, 3)])
def test_convolutions(nb, edge, cin, cout, k, stride, workspace):
    x, w, b = inputs.conv_i8_inputs(nb, edge, edge, cin, cout, k, k, seed=edge + cin + cout)
    want = oracle.conv2d_i8(x, w, b, stride, k // 2, 9, 1)
    nbytes = ops.ac_gemm_i8_workspace_bytes(want.size // cout, cout, k * k * cin) if workspace else 0
    out = torch.full(want.shape, 9, dtype=torch.int8, device="cuda")
    ops.ac_conv2d_i8(dev(x), dev(w), dev(b), out, stride, k // 2, 9, 1, workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
    np.testing.assert_array_equal(host(out), want)
