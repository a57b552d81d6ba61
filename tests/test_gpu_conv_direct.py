"""GPU parity of the convolution kernel for few channels (kernel rows of at most 32 bytes), bit for bit, where its forms change:
one and two chunks to a kernel row, windows that start on dwords, that do not, and that need the dword behind; every number of
K-steps; rows and columns of padding, tiles that touch no edge, one edge and the ends of the input; tiles that cross rows and
images; several tiles to a wave; column blocks of 32, 64 and 96 with partial columns; odd addresses, which it leaves to the others.
Which form each shape takes is asked on the host (test_conv_direct_loads.py)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu


def check(Nb, H, W, Cin, Cout, KH, KW, stride, pad, shift=8, act=1, offset=0, bias=True):
    x, w, b = inputs.conv_i8_inputs(Nb, H, W, Cin, Cout, KH, KW, seed=H * W + Cin + Cout)
    want = oracle.conv2d_i8(x, w, b if bias else np.zeros_like(b), stride, pad, shift, act)

    def put(a):  # `offset` bytes off an aligned address, zeros around it
        v = torch.zeros(a.size + 32, dtype=torch.int8, device="cuda")[offset:offset + a.size].view(a.shape)
        v.copy_(dev(a))
        return v

    out = put(np.full(want.shape, 17, np.int8))
    ops.ac_conv2d_i8(put(x), put(w), dev(b) if bias else None, out, stride, pad, shift, act)
    np.testing.assert_array_equal(host(out), want)


@pytest.mark.parametrize("Nb,H,W,Cin,Cout,KH,KW,stride,pad", [
    (2, 37, 40, 3, 64, 7, 7, 2, 3),     # two chunks of 13 bytes, seven K-steps
    (1, 33, 32, 4, 32, 7, 7, 1, 3),     # two chunks on dwords
    (1, 30, 31, 4, 40, 7, 7, 1, 3),     # ... the same, rows of 124 bytes
    (1, 41, 31, 5, 96, 6, 6, 1, 2),     # 30 bytes: the dword behind, six K-steps
    (2, 29, 33, 3, 48, 5, 5, 1, 2),     # one chunk of 15 bytes and the dword behind, three K-steps
    (2, 29, 33, 9, 17, 3, 3, 1, 1),     # 27 bytes, three K-steps
    (1, 26, 27, 8, 33, 4, 4, 2, 1),     # 32 bytes
    (2, 29, 33, 3, 80, 3, 3, 1, 1),     # one chunk, two K-steps, the second half beyond the kernel
    (1, 40, 44, 4, 16, 3, 3, 2, 1),     # ... on dwords
    (3, 50, 37, 1, 97, 8, 7, 1, 3),     # four K-steps of two rows, two column blocks
    (3, 21, 37, 1, 130, 5, 5, 1, 2),    # column blocks beyond the one they fill
    (2, 13, 19, 2, 1, 2, 8, 1, 4),      # one column
    (1, 9, 40, 13, 20, 5, 2, 1, 0),     # two chunks, five K-steps
    (1, 17, 23, 31, 64, 1, 1, 1, 0),    # single taps
    (1, 17, 23, 3, 64, 1, 1, 2, 0),
    (5, 16, 1, 17, 10, 4, 1, 1, 2),     # one column of pixels
    (3, 2, 6, 3, 8, 5, 5, 1, 2),        # images smaller than the kernel: every tile at an end of the input
    (1, 4, 4, 4, 17, 3, 3, 1, 1),       # rows of 16 bytes
    (1, 5, 5, 3, 17, 3, 3, 1, 1),       # ... and of 15
    (1, 6, 6, 3, 16, 3, 3, 1, 20),      # windows of padding only
    (11, 100, 101, 3, 48, 3, 3, 1, 1),  # several tiles to a wave
    (40, 61, 63, 3, 100, 1, 1, 1, 0),   # ... and two column blocks
    (1, 64, 64, 1, 16, 1, 16, 1, 0),    # the last window ends with the input, with and without the dword behind it
    (1, 16, 16, 2, 16, 8, 8, 1, 0),
    (1, 38, 38, 2, 16, 7, 7, 1, 3),     # ... in a tile that pads, the last but one of its rows
    (1, 2048, 15, 2, 16, 8, 7, 1, 3),
    (1, 1, 19, 1, 16, 1, 16, 1, 0),     # 19 bytes in all, left to another kernel, and 20
    (1, 1, 20, 1, 16, 1, 15, 1, 1),
])
def test_forms(Nb, H, W, Cin, Cout, KH, KW, stride, pad):
    check(Nb, H, W, Cin, Cout, KH, KW, stride, pad)
    check(Nb, H, W, Cin, Cout, KH, KW, stride, pad, offset=4, shift=17, act=0, bias=False)
    check(Nb, H, W, Cin, Cout, KH, KW, stride, pad, offset=1)  # an odd address: another kernel


@pytest.mark.parametrize("k,cin", [(1, 3), (3, 3), (3, 4), (5, 3), (5, 4), (7, 3), (7, 1)])
@pytest.mark.parametrize("edge", [32, 33, 35])
def test_edges_of_images(k, cin, edge):
    """Tiles of 32 pixels begin at every column of a row, and images at every pixel of a tile."""
    for stride in (1, 2):
        check(3, edge, edge + 1, cin, 16, k, k, stride, k // 2)
        check(2, edge, edge, cin, 24, k, k, stride, 0)
        check(2, edge, edge, cin, 24, k, k, stride, k)
