"""GPU parity of the 256 x 128 int8 tiles, whose bias row waits in LDS, and the 256 x 256 convolution tile, whose does not: no bias, a row at an
odd address, a matrix (products), columns beyond N, no K tile, one, fewer than the stages and many, several tiles to a
workgroup; bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu


def bias_of(b, kind):
    if kind == "none":
        return None, np.zeros_like(b)
    if kind == "odd":  # 4 bytes off an aligned address
        t = torch.zeros(b.size + 8, dtype=torch.int32, device="cuda")[1:1 + b.size]
        t.copy_(dev(b))
        return t, b
    return dev(b), b


@pytest.mark.parametrize("kind", ["odd", "none", "matrix"])
@pytest.mark.parametrize("M,N,K", [(256, 128, 0), (256, 128, 16), (250, 112, 128), (300, 144, 272), (257, 272, 400), (513, 48, 1040), (5000, 4112, 144)])
def test_products(M, N, K, kind):
    A, B, b = inputs.gemm_i8_inputs(M, N, K, seed=M + N + K, bias_matrix=kind == "matrix")
    t, b = bias_of(b, kind)
    C = torch.full((M, N), 9, dtype=torch.int8, device="cuda")
    At, Bt = (dev(A), dev(B)) if K else (torch.zeros((M, 16), dtype=torch.int8, device="cuda")[:, :0], torch.zeros((16, N), dtype=torch.int8, device="cuda")[:0])
    ops.ac_gemm_i8_planned(At, Bt, t, C, 8, 0, 192, 1)
    np.testing.assert_array_equal(host(C), oracle.gemm_i8(A, B, b, 8, 0))


@pytest.mark.parametrize("kind", ["odd", "none"])
@pytest.mark.parametrize("tile", [192, 256])
@pytest.mark.parametrize("Nb,H,W,Cin,Cout,k,stride,pad", [
    (1, 16, 16, 16, 128, 1, 2, 0), (2, 15, 13, 16, 272, 3, 1, 1), (1, 20, 19, 48, 144, 3, 2, 1), (1, 17, 33, 80, 256, 5, 1, 2), (70, 40, 41, 32, 304, 1, 1, 1)])
def test_convolutions(Nb, H, W, Cin, Cout, k, stride, pad, tile, kind):
    x, w, b = inputs.conv_i8_inputs(Nb, H, W, Cin, Cout, k, k, seed=H * W + Cout)
    t, b = bias_of(b, kind)
    want = oracle.conv2d_i8(x, w, b, stride, pad, 9, 0)
    out = torch.full(want.shape, 9, dtype=torch.int8, device="cuda")
    ops.ac_conv2d_i8(dev(x), dev(w), t, out, stride, pad, 9, 0, plan=(tile, 1))
    np.testing.assert_array_equal(host(out), want)
