// Which convolutions conv_i8_direct_kernel (conv_direct.hip) takes, in which form, and when its lanes may load a chunk from
// where it lies: host arithmetic without a HIP header, which the kernel shares and a test can compile by itself.
#pragma once
#include <stdint.h>

namespace ac {

// A load of 16 bytes a lane from any address costs a compute unit 65 clocks, from a dword 17 (from the L1, whatever the distance
// between lanes up to 32 bytes): a chunk comes from the dword its first byte lies in and is shifted into place.
enum ConvDirectShift {
  DIRECT_NONE,   // every chunk starts on a dword
  DIRECT_13,     // the dwords loaded hold 13 bytes of a chunk at least: that many of the run go to a chunk
  DIRECT_TAIL,   // 16, with the dword that follows
};
constexpr int conv_direct_payload(ConvDirectShift shift) { return shift == DIRECT_13 ? 13 : 16; }  // bytes of the run in a chunk
// Bytes from a chunk's first on that a load may reach.  The rounding down to a dword takes it no further: a chunk on a dword is
// read to its 16th or, with the dword that follows, its 20th byte.
constexpr int conv_direct_read(ConvDirectShift shift) { return shift == DIRECT_TAIL ? 20 : 16; }

// The pixel of a lane: first image row and first byte of the rows (either may lie outside the image), and the byte of the
// input at which its chunk of kernel row 0 would be.
struct ConvDirectWindow {
  int ih0, col, base;
};
// Nothing under the pixel is padding, and all that is loaded for it lies in the input.
constexpr bool conv_direct_whole(const ConvDirectWindow& w, int H, int KH, int RUN, int row_bytes, int a_bytes, int read) {
  return (w.ih0 >= 0) & (w.ih0 + KH <= H) & (w.col >= 0) & (w.col + RUN <= row_bytes) & (w.base + (KH - 1) * row_bytes + read <= a_bytes);
}
// The kernel rows first .. last lie inside the image, and their chunks, loaded from where they are, inside the input.
// (Lanes without such a row, and rows outside the image, load from the input's start, where conv_direct_form asks for
// `read` bytes.)  Otherwise every chunk of the tile is loaded from the nearest place at which 16 bytes exist, without a dword behind.
constexpr bool conv_direct_fits(const ConvDirectWindow& w, int first, int last, int row_bytes, int a_bytes, int read) {
  return (first > last) | ((w.base + first * row_bytes >= 0) & (w.base + last * row_bytes + read <= a_bytes));
}

// A convolution with a bias of at most a row; dword_base: the input's address is a multiple of 4.
struct ConvDirectCall {
  int32_t M, N, K, H, W, Cin, KH, KW, OH, OW, stride, pad, a_bytes, shift;
  bool dword_base;
};
struct ConvDirectForm {
  bool takes;
  bool narrow;  // a kernel row is one chunk, two rows to a K-step; otherwise two chunks
  ConvDirectShift shift;
  int nks, bn;  // K-steps, columns to a block
  int64_t n_blocks;
};
inline ConvDirectForm conv_direct_form(const ConvDirectCall& p) {
  const int64_t run = (int64_t)p.KW * p.Cin, w_bytes = (int64_t)p.K * p.N, lim = 1ll << 32;
  const bool dwords = (int64_t)p.stride * p.Cin % 4 == 0 && (int64_t)p.pad * p.Cin % 4 == 0 && (int64_t)p.W * p.Cin % 4 == 0;
  ConvDirectForm f = {};
  f.narrow = run <= 16;
  f.shift = dwords ? DIRECT_NONE : run <= 13 || (run > 16 && run <= 26) ? DIRECT_13 : DIRECT_TAIL;
  f.nks = f.narrow ? (p.KH + 1) / 2 : p.KH;
  if (run < 1 || run > 32 || f.nks < 1 || f.nks > (f.narrow ? 4 : 7) || p.a_bytes < conv_direct_read(f.shift) || w_bytes < 16 || w_bytes >= (1ll << 31) || p.N >= (1 << 29) || !p.dword_base) return f;
  if (p.shift < 1 || p.shift > 17) return f;  // (the rounding of the other shifts is not built into it)
  // Outputs beyond the caches are written in one moving window (3 x 3, 1 -> 96 channels on 31 images of 183 x 183, 100 MB, 33.9 us in
  // a run per XCD, 26.8 so; level below 40 MB), which the image kernel's workgroups in step do best where a pixel is one chunk
  // (1 x 1, 3 -> 96 on 22 of 222 x 222, 104 MB, 32.9 there and 39.1, on 20 of 176 x 176, 59 MB, 20.1 and 15.7).
  if (p.KH * p.KW == 1 && (int64_t)p.M * p.N > 90000000) return f;
  if (p.OW < 1 || (int64_t)p.M * p.OW >= lim || ((int64_t)p.M / p.OW + 1) * p.OH >= lim) return f;  // divisions by one multiply
  if ((int64_t)p.a_bytes + ((int64_t)p.KH + p.pad + 1) * ((int64_t)p.W + p.pad) * p.Cin >= 1ll << 31) return f;  // positions outside the image
  // the block width that computes the fewest columns beyond N
  auto cost = [&](int bn) { return (int64_t)((p.N + bn - 1) / bn) * (bn + 16); };
  f.bn = cost(96) <= cost(64) && cost(96) <= cost(32) ? 96 : (cost(64) <= cost(32) ? 64 : 32);
  f.n_blocks = ((int64_t)p.N + f.bn - 1) / f.bn;
  f.takes = f.n_blocks <= 65535;
  return f;
}

}  // namespace ac
