// int8 convolution of images whose channels are not whole 16-byte chunks (the first layer of a network, channel counts
// that are a multiple of nothing) for gfx950.
//
// A chunk of K of such a convolution starts at any byte of the image and may hang over two edges of its row, so the
// gather of gemm_ragged.hpp spends some forty instructions on every 16 bytes, for each output pixel anew, and that is
// what bounds it.  Here a workgroup owns 128 consecutive output pixels of one image and BN output channels, and copies
// the input rows under them into LDS once, 16 bytes a load wherever the row starts, with the padding columns and rows as
// zeros.  The KW * Cin bytes of a kernel row are contiguous under every pixel there, so K is walked as KH runs, each
// padded to whole chunks, and an MFMA operand is a 16-byte LDS read, shifted to its byte by the dword that follows (the
// bytes behind a run are the next pixel's and meet weight rows of zeros).  The weight rows (zero where K has no row) are
// copied as they are, K x BN, and read through the transposing loads; they are staged once for all units of the
// workgroup.
//
// A wave owns 32 pixels and the whole of BN: the work is staging and output stage, K is short, and one row tile per wave
// gives both the most waves.  Units of 256 pixels restage fewer rows and were never faster (7 x 7 stride 2 on 32 images
// of 224 x 224 x 3 25.4 us, 27.1 with 256).  96 columns to a wave need more than 128 registers: three waves to a SIMD
// and no spills (1 x 1, 1 -> 80 on 31 images of 152 x 152 22.6 us, with four and spills 56).
// Bound: latency where the output is small (staging, K loop and output stage of a unit follow one another; other
// workgroups of the compute unit and the early request of the next unit's rows overlap them), the instructions of
// staging and output stage where it is large.
//
// Against the any-alignment gather, against it with every pixel spread to whole dwords in LDS (four loads where this has
// one, longer runs), and now: 7 x 7 stride 2, 3 -> 64 channels on eight images of 224 x 224 30.6, 11.1, 10.5 us, on 32
// images 100, 28.8, 25.4; 1 x 1, 3 -> 64 on 22 images of 163 x 163 65, 17.2, 15.7; 5 x 5, 1 -> 80 on 16 of 113 x 113
// 17.1 and 11.8; 55 -> 58, 3 x 3 on four of 7 x 7 12.2 and 7.9.
#pragma once
#include <algorithm>
#include "gemm_ragged.hpp"

namespace ac {

constexpr int CONV_IMAGE_BM = 128;  // output pixels of a unit

struct ConvImageParams {
  int32_t L, PITCH;  // patch row: byte of the row's first pixel (a multiple of 16, the left padding before it), bytes
  int32_t CH;        // chunks of a patch row
  int32_t NC, RPI, p_row, p_c;  // staging: pieces of 64 chunks to a row; rows to a piece where a row is 32 chunks and less;
                                // from one piece of a wave to its next
  int32_t RUN, RUNP; // K bytes of one kernel row, and padded to whole chunks
  int32_t U, units;  // units per image, units
  int32_t patch;     // bytes of the patch, slack included
  int32_t w_bytes;   // bytes of the weights
  FastDiv dCH, dRUNP, dNC;
  unsigned u_magic, ow_magic;  // x / U and x / OW for units and pixels of an image by one multiply; 0: by a division
};

// DWORDS: every window starts on a dword of LDS.
template <int BN, bool DWORDS>
__global__ void __launch_bounds__(2 * CONV_IMAGE_BM) __attribute__((amdgpu_waves_per_eu(BN == 96 ? 3 : 4))) conv_i8_image_kernel(const GemmParams p, const ConvImageParams h, const int n_blocks) {
  using T = TypeI8;
  constexpr int BM = CONV_IMAGE_BM, THREADS = 2 * BM, TN = BN / 32, B_STRIDE = BN + 16, CPR = BN / 16, WB = 1024 / THREADS, PB = 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int* const bias = (int*)(smem + h.patch);
  unsigned char* const Bs = smem + h.patch + BN * 4;
  const int wgs = gridDim.x / n_blocks, wg = blockIdx.x / n_blocks;
  const int n0 = (blockIdx.x - wg * n_blocks) * BN;
  const int npix = p.OH * p.OW;
  const unsigned char* const weights = (const unsigned char*)p.B;

  struct Unit {
    int img, q0, ow0, ih0, rin;  // image, first pixel and its column, first input row, input rows
  };
  auto unit_of = [&](int u) {
    Unit w;
    w.img = h.u_magic ? (int)__umulhi((unsigned)u, h.u_magic) : u / h.U;
    w.q0 = (u - w.img * h.U) * BM;
    const int q_last = w.q0 + BM < npix ? w.q0 + BM - 1 : npix - 1;
    auto row_of = [&](int q) { return h.ow_magic ? (int)__umulhi((unsigned)q, h.ow_magic) : q / p.OW; };
    const int oh0 = row_of(w.q0);
    w.ow0 = w.q0 - oh0 * p.OW, w.ih0 = oh0 * p.stride - p.pad;
    w.rin = (row_of(q_last) - oh0) * p.stride + p.KH;
    return w;
  };
  // ---- the input rows of a unit.  A wave takes pieces wave, wave + 4, ...: 64 chunks of a row, or RPI short rows ----
  const int sub = h.RPI > 1 ? (int)h.dCH.div((unsigned)lane) : 0;
  const int j0 = lane - sub * h.CH;  // chunk of the row in piece 0
  const int row_bytes = p.W * p.Cin;
  struct Piece {
    int prow, c;  // piece row (RPI input rows) and piece of it
  };
  auto next_piece = [&](Piece& q) {
    q.prow += h.p_row, q.c += h.p_c;
    if (q.c >= h.NC) q.c -= h.NC, q.prow++;
  };
  v4i preg[PB];
  int pfix[PB];  // bytes by which the chunk was loaded early (the end of the input) | bytes of it inside the row << 8
  auto patch_load = [&](const Unit& w, Piece q) {
    const int img = w.img * p.H * row_bytes;  // (an input has fewer than 2^31 bytes)
    int jj = j0, ss = sub;
    asm volatile("" : "+v"(jj), "+v"(ss));  // the positions are computed afresh for every unit: kept, they fill the register file
#pragma unroll
    for (int i = 0; i < PB; i++) {
      if (q.prow * h.RPI >= w.rin) break;  // (wave-uniform; small patches have one or two pieces to a wave)
      const int b = (jj + q.c * 64) * 16 - h.L;
      const int ih = w.ih0 + q.prow * h.RPI + ss;
      const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)b < (unsigned)row_bytes;
      const int valid = row_bytes - b < 16 ? row_bytes - b : 16;
      int g = img + __mul24(ih, row_bytes) + b;
      g = in ? g : 0;
      const int a = g < p.a_bytes - 16 ? g : p.a_bytes - 16;  // (the launcher makes sure that there are 16 bytes)
      preg[i] = load16_any((const unsigned char*)p.A + (unsigned)a);
      pfix[i] = in ? (g - a) | (valid << 8) : 0;
      next_piece(q);
    }
  };
  auto patch_store = [&](const Unit& w, Piece q) {
    int jj = j0, ss = sub;
    asm volatile("" : "+v"(jj), "+v"(ss));
    if (ss >= h.RPI) ss = 1 << 20;
#pragma unroll
    for (int i = 0; i < PB; i++) {
      if (q.prow * h.RPI >= w.rin) break;
      const int row = q.prow * h.RPI + ss, j = jj + q.c * 64;
      v4i v = preg[i];
#pragma unroll
      for (int e = 0; e < 4; e++) v[e] = pfix[i] ? v[e] : 0;  // padding
      if (pfix[i] != 0 && pfix[i] != 16 << 8) v = chunk_apply<false>(v, chunk_fix(pfix[i] & 255, 0, pfix[i] >> 8));  // the row's end
      if (row < w.rin && j < h.CH) *(v4i*)(smem + __mul24(row, h.PITCH) + 16 * j) = v;
      next_piece(q);
    }
    return q;
  };
  Piece piece0;
  piece0.prow = (int)h.dNC.div((unsigned)wave), piece0.c = wave - piece0.prow * h.NC;
  // ---- weights: all kernel rows as nrow K rows (whole K-steps of 32), WB chunks per thread at a time ----
  const int nks = (p.KH * h.RUNP + 31) >> 5, nrow = nks * 32;
  v4i wreg[WB];
  int wover[WB];  // bytes by which a chunk was loaded early (the end of the weights); 16: nothing of it is kept
  auto weights_load = [&](int base) {
#pragma unroll
    for (int i = 0; i < WB; i++) {
      const int idx = base + i * THREADS + t;
      const int k = idx / CPR, cc = idx - k * CPR;
      const int kh = (int)h.dRUNP.div((unsigned)k), r = k - kh * h.RUNP;
      const int col = n0 + cc * 16;
      const bool in = kh < p.KH && r < h.RUN && col < p.N;
      int g = (kh * h.RUN + r) * p.N + col;
      g = in ? g : 0;
      const int q = g < h.w_bytes - 16 ? g : h.w_bytes - 16;
      wreg[i] = load16_any(weights + (unsigned)q);
      wover[i] = in ? g - q : 16;
    }
  };
  auto weights_store = [&](int base) {
#pragma unroll
    for (int i = 0; i < WB; i++) {
      const int idx = base + i * THREADS + t;
      const int k = idx / CPR, cc = idx - k * CPR;
      v4i v = wreg[i];
      if (p.N % 16 != 0 && wover[i] != 0) v = chunk_apply<false>(v, chunk_fix(wover[i] & 15, 0, 16));
#pragma unroll
      for (int e = 0; e < 4; e++) v[e] = wover[i] == 16 ? 0 : v[e];
      if (k < nrow) *(v4i*)(Bs + k * B_STRIDE + cc * 16) = v;
    }
  };
  Unit w = unit_of(wg);  // (there are no more workgroups to a column block than units)
  // everything is requested before anything is waited for
  weights_load(0);
  const int my_bias = p.bias && t < BN && n0 + t < p.N ? p.bias[n0 + t] : 0;
  patch_load(w, piece0);
  weights_store(0);
#pragma unroll 1
  for (int base = WB * THREADS; base < nrow * CPR; base += WB * THREADS) {
    weights_load(base);
    weights_store(base);
  }
  if (t < BN) bias[t] = my_bias;

#pragma unroll 1
  for (int u = wg; u < h.units; u += wgs) {
    Piece q = patch_store(w, piece0);
#pragma unroll 1
    while (q.prow * h.RPI < w.rin) {
      patch_load(w, q);
      q = patch_store(w, q);
    }
    // this lane's pixel (beyond the image: the last one) and the first byte of its window
    const int qi = w.q0 + wave * 32 + (lane & 31);
    const int x = w.ow0 + (qi < npix ? qi : npix - 1) - w.q0;
    const int pr = (int)p.dOW.div((unsigned)x), pc = x - pr * p.OW;
    const int win = (pr * h.PITCH + pc * p.Cin) * p.stride + h.L - p.pad * p.Cin;
    const int pix = DWORDS ? win : win & ~3, shift = win & 3;  // patch rows and chunks of K keep the byte inside the dword

    typename T::accv acc[TN];
    const Unit cur = w;
    block_sync();
    if (u + wgs < h.units) {  // the next unit's first rows are under way while this one is multiplied and stored
      w = unit_of(u + wgs);
      patch_load(w, piece0);
    }
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const v4i b4 = *(const v4i*)(bias + 32 * j + 8 * q + 4 * half);
#pragma unroll
        for (int e = 0; e < 4; e++) acc[j][4 * q + e] = b4[e];
      }
    // chunk 2 ks + half of the walk: kernel row and byte r of its run
    const int dkh = h.RUNP == 16 ? 2 : (h.RUNP == 32 ? 1 : 0), dr = 32 - dkh * h.RUNP, step = dkh * h.PITCH + dr, wrap = h.PITCH - h.RUNP;
    int r = half * 16, off = pix + r;
    if (r >= h.RUNP) r -= h.RUNP, off += wrap;
    const unsigned char* bp = Bs + (half * 16 + ((lane & 15) >> 1)) * B_STRIDE + 16 * ((lane >> 4) & 1) + 8 * (lane & 1);
    v4i a[2], b[2][TN];
    int a4[2];  // the dword that follows
    auto read = [&](int s) {
      a[s] = ((const Dwords16*)(smem + off))->v;
      if constexpr (!DWORDS) a4[s] = *(const int*)(smem + off + 16);
      off += step, r += dr;
      if (r >= h.RUNP) r -= h.RUNP, off += wrap;
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, bp + 32 * j));
        const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, bp + 32 * j + 8 * B_STRIDE));
        b[s][j] = (v4i){lo[0], lo[1], hi[0], hi[1]};
      }
      bp += 32 * B_STRIDE;
    };
    auto multiply = [&](int s) {
      if constexpr (!DWORDS) {
        const v4i w4 = a[s];
#pragma unroll
        for (int e = 0; e < 4; e++) a[s][e] = (int)__builtin_amdgcn_alignbyte((unsigned)(e < 3 ? w4[e + 1] : a4[s]), (unsigned)w4[e], (unsigned)shift);
      }
#pragma unroll
      for (int j = 0; j < TN; j++) acc[j] = T::mfma(b[s][j], a[s], acc[j]);
    };
    read(0);
    int ks = 0;
#pragma unroll 1
    for (; ks + 2 < nks; ks += 2) {
      read(1);
      multiply(0);
      read(0);
      multiply(1);
    }
    if (ks + 1 < nks) {
      read(1);
      multiply(0);
      multiply(1);
    } else {
      multiply(0);
    }
    block_sync();  // the patch may be overwritten

    // ---- output stage: a lane holds 16 consecutive columns of its pixel after the exchange ----
    int8_t* const row = (int8_t*)p.C + ((int64_t)cur.img * npix + qi) * p.ldc;
    const EpilogueI8::FastQuant f = EpilogueI8::fast_quant(p.shift, p.act);
#pragma unroll
    for (int j = 0; j < TN; j++) {
      if (n0 + 32 * j >= p.N) break;
      int v[16];
#pragma unroll
      for (int e = 0; e < 16; e++) v[e] = acc[j][e];
      const v4i o = EpilogueI8::quant16<true>(v, f);
      const int n = n0 + 32 * j + 16 * half;
      if (qi < npix) store_run16(row + n, o, p.N - n);
      __builtin_amdgcn_sched_barrier(0);  // one column tile at a time: interleaved, the values of all of them spill
    }
  }
}

// Geometry for column blocks of bn, or false when the convolution does not fit (its input rows
// or the weights of one kernel row are too large for LDS).
static inline bool conv_image_plan(const GemmParams& p, int bn, ConvImageParams* h, size_t* lds) {
  const int bm = CONV_IMAGE_BM;
  const int64_t w_bytes = (int64_t)p.K * p.N, npix = (int64_t)p.OH * p.OW;
  if (p.Cin < 1 || p.KH < 1 || p.KW < 1 || npix < 1 || npix >= (1ll << 31) || p.M % npix != 0 || p.a_bytes < 16 || w_bytes < 16 || w_bytes >= (1ll << 31) || p.N >= (1 << 29)) return false;
  if ((p.bias != nullptr && p.bias_ld != 0) || p.shift < 1 || p.shift > 17) return false;  // (the rounding of the other shifts is not built into it)
  if ((int64_t)p.W * p.Cin >= (1 << 23)) return false;  // 24-bit products
  const int64_t run = (int64_t)p.KW * p.Cin, runp = (run + 15) / 16 * 16, left = ((int64_t)p.pad * p.Cin + 15) / 16 * 16;
  // the last window of a row, its padding to whole chunks and the dword that follows
  const int64_t pitch = (left - (int64_t)p.pad * p.Cin + (int64_t)(p.OW - 1) * p.stride * p.Cin + runp + 4 + 15) / 16 * 16;
  const int64_t span = std::min<int64_t>((bm + p.OW - 2) / p.OW + 1, p.OH);  // output rows that bm consecutive pixels can touch
  const int64_t rin = (span - 1) * p.stride + p.KH, budget = 160 * 1024;
  // one row and one chunk of slack: the reads of the padding of a run, and of an odd last chunk
  const int64_t patch = (rin + 1) * pitch + 32;
  if (runp > 32768 || pitch > budget || patch > budget) return false;
  const int64_t need = patch + bn * 4 + (p.KH * runp + 31) / 32 * 32 * (bn + 16);
  if (need > budget) return false;
  const int64_t units_per_image = (npix + bm - 1) / bm, units = p.M / npix * units_per_image;
  if (units > (1 << 30)) return false;
  h->L = (int32_t)left, h->PITCH = (int32_t)pitch, h->CH = (int32_t)(pitch / 16), h->RUN = (int32_t)run, h->RUNP = (int32_t)runp;
  h->U = (int32_t)units_per_image, h->units = (int32_t)units, h->patch = (int32_t)patch, h->w_bytes = (int32_t)w_bytes;
  h->NC = (h->CH + 63) / 64, h->RPI = h->CH <= 32 ? 64 / h->CH : 1;
  h->p_row = bm / 32 / h->NC, h->p_c = bm / 32 - h->p_row * h->NC;
  h->u_magic = units * units_per_image < (1ll << 32) ? FastDiv::make(h->U).magic : 0;
  h->ow_magic = npix * p.OW < (1ll << 32) ? FastDiv::make(p.OW).magic : 0;
  h->dCH = FastDiv::make(h->CH), h->dNC = FastDiv::make(h->NC), h->dRUNP = FastDiv::make(h->RUNP);
  *lds = (size_t)need;
  return true;
}

template <int BN, bool DWORDS>
static hipError_t launch_conv_image_form(const GemmParams& p, const ConvImageParams& h, size_t lds, hipStream_t stream) {
  auto kern = conv_i8_image_kernel<BN, DWORDS>;
  static std::atomic<bool> configured{false};
  if (const hipError_t e = allow_dynamic_lds_once(configured, kern, 160 * 1024)) return e;
  const int n_blocks = (p.N + BN - 1) / BN;
  // workgroups resident on a compute unit: by LDS, and by registers (four waves to a SIMD, three of 96 columns)
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(160 * 1024 / (int64_t)lds, BN == 96 ? 3 : 4));
  int64_t wgs = per_cu * compute_units() / n_blocks;
  if (wgs < 1) wgs = 1;
  if (wgs > h.units) wgs = h.units;
  return launch_kernel(kern, dim3((unsigned)(wgs * n_blocks)), dim3(2 * CONV_IMAGE_BM), lds, stream, p, h, n_blocks);
}

template <int BN>
static hipError_t launch_conv_image_kernel(const GemmParams& p, const ConvImageParams& h, size_t lds, hipStream_t stream) {
  const bool dwords = (int64_t)p.stride * p.Cin % 4 == 0 && (int64_t)p.pad * p.Cin % 4 == 0;
  return dwords ? launch_conv_image_form<BN, true>(p, h, lds, stream) : launch_conv_image_form<BN, false>(p, h, lds, stream);
}

// Whether a convolution of sixteen channels, which the direct-to-LDS gather takes too, belongs here: it copies every input
// row under a unit whole, so not where most of a row lies beside the unit's pixels or between its windows (1 x 3 on rows
// of 1000 pixels 31.8 us on the gather and 34.9 here, 9 x 1 stride 3 on rows of 280 39 and 78: patches of 31 and 66 KB;
// 2 x 2 stride 3 6.8 and 7.4), nor where less than half of a unit exists (16 -> 512 on 512 images of 7 x 7 12.5 and 15.1).
// Elsewhere 3 x 3 kernels over 16 channels: 16 -> 64 on 32 images of 56 x 56 10.9 us tiled and 7.2 here, 16 -> 320 on 50 of
// 50 x 50 35.9 and 19.5, stride 2, 16 -> 320 on 55 of 84 x 131 42 and 30.
// Kernels between nine taps and more than 32 stay with the gather; beyond it has twice the rows and a few columns leave
// it idle (7 x 7, 16 -> 16 on 64 images of 28 x 28 13.4 and 6.9, 6 x 6, 16 -> 48 on 4384 tiles 2.4 times its rate).
static inline bool conv_image_takes_sixteen(const GemmParams& p) {
  const int taps = p.KH * p.KW;
  if (p.Cin != 16 || p.stride > 2 || taps < 2 || (taps > 9 && (taps <= 32 || p.N > 64))) return false;
  ConvImageParams h;
  size_t lds = 0;
  return conv_image_plan(p, 32, &h, &lds) && h.patch <= 28 * 1024 && 2 * (int64_t)p.OH * p.OW >= (int64_t)h.U * CONV_IMAGE_BM;
}

// Launches the kernel when it takes the convolution and is the faster one; false otherwise.
static inline bool launch_conv_image(const GemmParams& p, hipStream_t stream, hipError_t* e) {
  // the block width that computes the fewest columns beyond N
  auto cost = [&](int bn) { return (int64_t)((p.N + bn - 1) / bn) * (bn + 16); };
  const int bn = cost(96) <= cost(64) && cost(96) <= cost(32) ? 96 : (cost(64) <= cost(32) ? 64 : 32);
  ConvImageParams h;
  size_t lds = 0;
  if (!conv_image_plan(p, bn, &h, &lds)) return false;
  // A single tap reuses nothing of the patch and is a plain product, for which the any-alignment GEMM has whole chunks
  // from 64 channels on (60 -> 60 channels on 256 images of 14 x 14 9.6 us there and 6.9 here, 130 -> 100 on eight 6.1
  // and 7.9, 512 -> 250 7.4 and 17.9).  From 64 K-steps on the weights of a block are most of the work, and a
  // workgroup has them to itself (51 -> 28 channels, 7 x 7 on three images of 19 x 19, 81 K-steps: 13.7 us cut along K
  // there, 20 here; 40 -> 20, 7 x 7 on eight of 56 x 56, 63 K-steps: 28 and 18).
  if (p.KH * h.RUNP > 64 * 32 || (p.KH * p.KW == 1 && p.Cin > 64)) return false;
  *e = bn == 96 ? launch_conv_image_kernel<96>(p, h, lds, stream) : bn == 64 ? launch_conv_image_kernel<64>(p, h, lds, stream) : launch_conv_image_kernel<32>(p, h, lds, stream);
  return true;
}

}  // namespace ac
