"""The convolution kernel for few channels, on the host: the forms that the shapes of its GPU tests take, and its loads.  For every form, kernel, stride and padding over small
images, what each lane requests of the input lies inside the input (the kernel's own conditions, its positions replayed)."""
import ctypes
import os
import subprocess

import pytest

import test_gpu_conv_direct as gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_18574_amd", "csrc")
SHIM = """
#include "conv_direct_rules.hpp"
using namespace ac;
static ConvDirectCall call_of(int Nb, int H, int W, int Cin, int N, int KH, int KW, int stride, int pad) {
  const int OH = (H + 2 * pad - KH) / stride + 1, OW = (W + 2 * pad - KW) / stride + 1;
  return {Nb * OH * OW, N, KH * KW * Cin, H, W, Cin, KH, KW, OH, OW, stride, pad, Nb * H * W * Cin, 8, true};
}
extern "C" int form(int Nb, int H, int W, int Cin, int N, int KH, int KW, int stride, int pad) {
  const ConvDirectForm f = conv_direct_form(call_of(Nb, H, W, Cin, N, KH, KW, stride, pad));
  return f.takes ? (f.narrow ? 1000 : 0) + 100 * f.shift + f.nks : -1;
}
extern "C" int columns(int N) { return conv_direct_form(call_of(2, 29, 33, 3, N, 3, 3, 1, 1)).bn; }
extern "C" int takes(int shift, int dword_base) {
  ConvDirectCall c = call_of(2, 29, 33, 3, 16, 3, 3, 1, 1);
  c.shift = shift, c.dword_base = dword_base != 0;
  return conv_direct_form(c).takes;
}
// The most bytes that a load reaches beyond the input (before its start: as a negative number), over all tiles, lanes and K-steps; -1000000:
// not taken.  kinds[0 .. 2]: tiles loaded whole, in part, and at an end of the input.
extern "C" int beyond(int Nb, int H, int W, int Cin, int N, int KH, int KW, int stride, int pad, int* kinds) {
  const ConvDirectCall c = call_of(Nb, H, W, Cin, N, KH, KW, stride, pad);
  const ConvDirectForm f = conv_direct_form(c);
  if (!f.takes) return -1000000;
  const int read = conv_direct_read(f.shift), payload = conv_direct_payload(f.shift), row_bytes = W * Cin, RUN = KW * Cin;
  int worst = 0;
  for (int tile = 0; tile * 32 < c.M; tile++) {
    ConvDirectWindow w[64];
    int first[64], last[64];
    bool whole = true, near = false;
    for (int lane = 0; lane < 64; lane++) {
      int m = tile * 32 + lane % 32;
      m = m < c.M ? m : c.M - 1;
      const int q = m / c.OW, ow = m % c.OW, img = q / c.OH, oh = q % c.OH;
      const int ih0 = oh * stride - pad, col = (ow * stride - pad) * Cin;
      w[lane] = {ih0, col, (img * H + ih0) * row_bytes + col + (f.narrow ? 0 : payload * (lane / 32))};
      first[lane] = ih0 < 0 ? -ih0 : 0, last[lane] = H - 1 - ih0 < KH - 1 ? H - 1 - ih0 : KH - 1;
      whole &= conv_direct_whole(w[lane], H, KH, RUN, row_bytes, c.a_bytes, read);
      near |= !conv_direct_fits(w[lane], first[lane], last[lane], row_bytes, c.a_bytes, read);
    }
    kinds[whole ? 0 : near ? 2 : 1]++;
    for (int lane = 0; lane < 64; lane++)
      for (int ks = 0; ks < f.nks; ks++) {
        int kh = f.narrow ? 2 * ks + lane / 32 : ks, g;
        if (whole && ks == f.nks - 1 && kh >= KH) kh = KH - 1;
        if (whole) g = w[lane].base + kh * row_bytes;
        else g = kh >= first[lane] && kh <= last[lane] ? w[lane].base + kh * row_bytes : 0;
        int bytes = 16;
        if (!whole && near) g = g < 0 ? 0 : g > c.a_bytes - 16 ? c.a_bytes - 16 : g;
        else if (f.shift != DIRECT_NONE) g &= ~3, bytes = f.shift == DIRECT_TAIL ? 20 : 16;
        if (g < 0) return g;
        if (g + bytes - c.a_bytes > worst) worst = g + bytes - c.a_bytes;
      }
  }
  return worst;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    folder = tmp_path_factory.mktemp("direct")
    (folder / "shim.cpp").write_text(SHIM)
    so = str(folder / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", so, str(folder / "shim.cpp")], check=True)
    return ctypes.CDLL(so)


NARROW, BYTES_13, TAIL = 1000, 100, 200  # + K-steps


def test_forms_of_the_gpu_tests(rules):
    shapes = next(m.args[1] for m in gpu.test_forms.pytestmark if m.name == "parametrize")
    assert [rules.form(*s) for s in shapes] == [
        BYTES_13 + 7, 7, 7, TAIL + 6, NARROW + TAIL + 3, TAIL + 3, 4, NARROW + BYTES_13 + 2, NARROW + 2, NARROW + BYTES_13 + 4, NARROW + BYTES_13 + 3, NARROW + TAIL + 1, BYTES_13 + 5,
        TAIL + 1, NARROW + BYTES_13 + 1, BYTES_13 + 4, NARROW + TAIL + 3, NARROW + 2, NARROW + BYTES_13 + 2, NARROW + BYTES_13 + 2, NARROW + BYTES_13 + 2, NARROW + BYTES_13 + 1,
        NARROW + TAIL + 1, NARROW + TAIL + 4, NARROW + TAIL + 4, NARROW + TAIL + 4, -1, NARROW + TAIL + 1]
    for m in gpu.test_edges_of_images.pytestmark:
        if m.args[0] == "k,cin":
            assert all(rules.form(2, edge, edge, cin, 24, k, k, 1, pad) > 0 for k, cin in m.args[1] for edge in (32, 33, 35) for pad in (0, k // 2, k))
    assert [rules.columns(n) for n in (1, 32, 33, 64, 80, 96, 97, 130, 192)] == [32, 32, 64, 64, 96, 96, 64, 96, 96]


def test_calls_left_to_the_others(rules):
    assert [rules.takes(shift, 1) for shift in (0, 1, 17, 18)] == [0, 1, 1, 0] and not rules.takes(8, 0)
    # 33 bytes to a kernel row, nine rows, eight of two chunks, a single tap on 189 MB of output, inputs of 15 bytes and, with the dword behind, 19
    for shape in [(2, 40, 40, 11, 16, 3, 3, 1, 1), (2, 40, 40, 3, 16, 9, 3, 1, 1), (2, 40, 40, 6, 16, 8, 3, 1, 1), (40, 222, 222, 3, 96, 1, 1, 1, 0),
                  (1, 1, 15, 1, 16, 1, 1, 1, 0), (1, 1, 19, 1, 16, 1, 16, 1, 0)]:
        assert rules.form(*shape) == -1, shape
    assert rules.form(1, 2, 4, 2, 16, 1, 1, 1, 0) > 0 and rules.form(1, 1, 16, 1, 16, 1, 1, 1, 0) > 0


def check(rules, shape, kinds):
    beyond = rules.beyond(*shape, kinds)
    assert beyond in (0, -1000000), (shape, beyond)
    return beyond == 0


@pytest.mark.parametrize("shape", [
    (1, 64, 64, 1, 16, 1, 16, 1, 0), (1, 64, 64, 2, 16, 2, 8, 1, 0), (1, 16, 32, 1, 16, 8, 16, 1, 0), (1, 2048, 15, 2, 16, 8, 7, 1, 3),  # the last chunk ends with the input
    (1, 16, 16, 2, 16, 8, 8, 1, 0), (1, 32, 32, 1, 16, 8, 16, 1, 0), (1, 38, 38, 2, 16, 7, 7, 1, 3), (2, 20, 20, 2, 16, 7, 7, 1, 3)])
def test_chunks_that_end_with_the_input(rules, shape):
    kinds = (ctypes.c_int * 3)()
    assert check(rules, shape, kinds)


def test_inputs_of_a_few_bytes(rules):
    kinds = (ctypes.c_int * 3)()
    for W in range(1, 25):
        for KW in range(1, 17):
            for pad in (0, 1, 8):
                if KW <= W + 2 * pad:
                    check(rules, (1, 1, W, 1, 16, 1, KW, 1, pad), kinds)


def test_every_form(rules):
    kinds, forms = (ctypes.c_int * 3)(), set()
    for run in range(1, 33):
        for Cin in (c for c in range(1, run + 1) if run % c == 0):
            KW = run // Cin
            for KH in range(1, 8 if run > 16 else 9):
                for H, W in ((1, 16), (5, 5), (9, 8), (16, 21), (3, 40)):
                    for stride in (1, 2, 3):
                        for pad in sorted({0, 1, KH // 2, KW // 2, KW, KW + 4}):
                            if KH > H + 2 * pad or KW > W + 2 * pad:
                                continue
                            for Nb in (1, 3):
                                if check(rules, (Nb, H, W, Cin, 16, KH, KW, stride, pad), kinds):
                                    forms.add(rules.form(Nb, H, W, Cin, 16, KH, KW, stride, pad))
    # one chunk to a kernel row: one to four K-steps, two chunks: one to seven, each on dwords, with 13 bytes to a chunk and with the dword behind
    assert forms == {1000 + 100 * s + n for s in range(3) for n in range(1, 5)} | {100 * s + n for s in range(3) for n in range(1, 8)}
    assert all(kinds), list(kinds)
