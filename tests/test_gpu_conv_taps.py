"""GPU parity of convolutions of more than 32 kernel taps whose channels are whole 16-byte chunks (the direct-to-LDS
gather, one validity bit per kernel row and column), bit for bit: windows over every edge, kernels of 32 rows and
columns (the most one bit each can say), of 33 columns (any-alignment kernel), with and without a cut K range."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Nb,H,W,Cin,Cout,KH,KW,stride,pad", [
    (1, 20, 20, 16, 32, 7, 7, 1, 3),
    (3, 9, 9, 32, 48, 7, 7, 1, 3),       # every window hangs over two edges
    (2, 21, 17, 16, 16, 6, 6, 1, 2),     # K = 576: one wave per tile
    (1, 14, 13, 16, 80, 8, 8, 2, 4),     # K = 1024
    (1, 40, 37, 16, 16, 32, 32, 1, 5),   # the last bit of both masks
    (1, 40, 37, 16, 16, 2, 32, 3, 31),   # windows of padding only
    (1, 8, 60, 16, 32, 2, 33, 1, 0),     # a kernel column beyond the masks
    (2, 2, 2, 32, 16, 7, 7, 1, 3),       # an image smaller than the kernel
    (12, 40, 41, 16, 272, 7, 7, 1, 3),   # more tiles than one round
    (5, 61, 61, 32, 144, 6, 6, 1, 3),    # ... whose plan is weight-stationary: the tile by the estimates
])
def test_many_taps(Nb, H, W, Cin, Cout, KH, KW, stride, pad):
    x, w, b = inputs.conv_i8_inputs(Nb, H, W, Cin, Cout, KH, KW, seed=H * W + Cin)
    want = oracle.conv2d_i8(x, w, b, stride, pad, 10, 1)
    nbytes = ops.ac_gemm_i8_workspace_bytes(want.shape[0] * want.shape[1] * want.shape[2], Cout, KH * KW * Cin)
    for ws in (None, torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None):
        out = torch.full(want.shape, 17, dtype=torch.int8, device="cuda")
        ops.ac_conv2d_i8(dev(x), dev(w), dev(b), out, stride, pad, 10, 1, workspace=ws)
        np.testing.assert_array_equal(host(out), want)
