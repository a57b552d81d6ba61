"""GPU parity of the convolution kernel for channels that are not whole 16-byte chunks, bit for bit, where its forms
change: windows that start on any byte of a dword, runs of one chunk, two and more, odd and even K-steps, patches of one
piece to a wave and of many, short rows that share a piece, rows that end inside a chunk, units that end inside an image,
column blocks of 32, 64 and 96 with partial columns, weights and inputs that end inside a chunk, odd addresses."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from paper_2505_18574_amd import inputs, ops

pytestmark = pytest.mark.gpu


def odd(a):
    """A dense copy that starts one byte off an aligned address."""
    buf = torch.zeros(a.size + 16, dtype=torch.int8, device="cuda")
    v = buf[1:1 + a.size].view(a.shape)
    v.copy_(dev(a))
    return v


def check(Nb, H, W, Cin, Cout, KH, KW, stride, pad, shift=8, act=1, put=dev, bias=True):
    x, w, b = inputs.conv_i8_inputs(Nb, H, W, Cin, Cout, KH, KW, seed=H * W + Cin)
    want = oracle.conv2d_i8(x, w, b if bias else np.zeros_like(b), stride, pad, shift, act)
    out = put(np.full(want.shape, 17, np.int8))
    ops.ac_conv2d_i8(put(x), put(w), dev(b) if bias else None, out, stride, pad, shift, act)
    np.testing.assert_array_equal(host(out), want)


@pytest.mark.parametrize("Nb,H,W,Cin,Cout,KH,KW,stride,pad", [
    (2, 40, 37, 3, 64, 7, 7, 2, 3),      # seven runs of two chunks, an odd number of K-steps
    (1, 30, 31, 1, 16, 3, 3, 1, 1),      # three runs of one chunk: the last K-step is half beyond K
    (1, 30, 31, 2, 96, 2, 4, 1, 2),      # two runs of one chunk: one K-step
    (3, 1, 1, 3, 8, 5, 5, 1, 2),         # images of three bytes, all but one tap padding
    (5, 7, 7, 14, 27, 3, 3, 1, 1),       # short rows share a piece; 27 columns
    (1, 5, 3, 1, 16, 3, 3, 1, 1),        # an input of 15 bytes: not taken
    (1, 4, 4, 1, 17, 3, 3, 1, 1),        # ... of 16
    (1, 17, 1, 1, 17, 3, 1, 1, 0),       # ... of 17, rows of one byte
    (2, 9, 1100, 2, 40, 3, 3, 2, 1),     # rows of more than 64 chunks
    (2, 13, 11, 59, 57, 3, 3, 1, 1),     # runs of 177 bytes
    (1, 9, 200, 5, 130, 3, 3, 1, 1),     # several pieces to a row, two column blocks, the second partial
    (2, 33, 1, 3, 33, 3, 1, 2, 0),       # one column of pixels
    (1, 1, 300, 6, 70, 1, 5, 3, 1),      # one row
    (9, 12, 11, 3, 97, 3, 3, 1, 1),      # 97 columns: blocks beyond the one they fill
    (1, 70, 70, 4, 1, 1, 1, 1, 0),       # a plain product, one column
    (2, 17, 16, 64, 50, 1, 1, 2, 0),     # the widest single tap taken
    (2, 17, 16, 65, 50, 1, 1, 2, 0),     # ... and the first not taken
    (1, 18, 18, 40, 20, 7, 7, 1, 3),     # 63 K-steps
    (1, 18, 18, 41, 20, 7, 7, 1, 3),     # beyond 64: the any-alignment kernel
    (8, 100, 101, 3, 48, 7, 7, 2, 3),    # several units to a workgroup
    (13, 57, 59, 16, 32, 3, 3, 1, 1),    # sixteen channels, more than 512 tiles
    (1, 6, 6, 3, 16, 3, 3, 1, 20),       # windows of padding only
])
def test_forms(Nb, H, W, Cin, Cout, KH, KW, stride, pad):
    check(Nb, H, W, Cin, Cout, KH, KW, stride, pad)
    check(Nb, H, W, Cin, Cout, KH, KW, stride, pad, put=odd, bias=False)


@pytest.mark.parametrize("shift,act", [(0, 0), (1, 0), (17, 0), (17, 1), (18, 0), (31, 1)])
def test_shifts(shift, act):
    check(2, 15, 16, 3, 36, 3, 3, 1, 1, shift, act)


@pytest.mark.parametrize("Nb,H,W,Cout,KH,KW,stride,pad", [
    (13, 57, 59, 48, 3, 3, 2, 1),     # fewer than 512 tiles: the gather
    (50, 57, 59, 48, 3, 3, 2, 1),     # ... more: here
    (50, 57, 59, 48, 3, 3, 3, 1),     # stride 3: the gather
    (700, 7, 7, 64, 3, 3, 1, 1),      # units less than half full: the gather
    (500, 9, 9, 80, 3, 3, 1, 1),      # ... and more than half
    (2, 40, 1000, 32, 1, 3, 1, 0),    # a patch of 32 KB: the gather
    (2, 70, 500, 32, 1, 3, 1, 0),     # ... of 16: here
    (36, 31, 33, 64, 7, 7, 1, 3),     # 49 taps and 64 columns: here
    (36, 31, 33, 80, 7, 7, 1, 3),     # ... and 80: the gather
    (40, 31, 33, 64, 2, 5, 1, 1),     # ten taps: the gather
    (111, 14, 74, 32, 2, 4, 2, 0),    # one wave per tile
])
def test_sixteen_channels(Nb, H, W, Cout, KH, KW, stride, pad):
    """Both sides of the rule that shares the convolutions of sixteen channels out."""
    check(Nb, H, W, 16, Cout, KH, KW, stride, pad)


def test_unit_order_and_many_units():
    """More units than workgroups: every workgroup walks over several, requesting the next one's rows early."""
    check(37, 50, 49, 3, 64, 3, 3, 1, 1)
    check(64, 60, 61, 1, 33, 1, 1, 1, 0)
