// int8 convolution of images whose channels are not whole 16-byte chunks (the first layer of a network, channel counts
// that are a multiple of nothing) for gfx950.
//
// A chunk of K of such a convolution starts at any byte of the image and may hang over two edges of its row, so the
// gather of gemm_ragged.hpp spends some forty instructions on every 16 bytes, for each output pixel anew, and that is
// what bounds it.  Here a workgroup owns BM consecutive output pixels of one image and BN output channels, and lays the
// input rows under them out in LDS once: pixels spread to CP = Cin rounded up to whole dwords, padding columns and rows
// as zeros.  One dword of a pixel is one unaligned load, wherever the pixel starts; the bytes behind its last channel
// are the next pixel's and meet weight rows of zeros.  The KW * CP bytes of a kernel row are then contiguous under every
// pixel, so K is walked as KH runs, each padded to whole chunks, and an MFMA operand is a 16-byte LDS read with no
// mask.  The weight rows (zero where K has no row) are copied as they are, K x BN, and read through the transposing
// loads; they are staged once for all units of the workgroup.
//
// A wave owns 32 pixels and the whole of BN: the work is staging and output stage, K is short, and one row tile per wave
// gives both the most waves.  Bound: latency where the output is small (staging, K loop and output stage of a unit follow
// one another; other workgroups of the compute unit and the early request of the next unit's rows overlap them), the
// instructions of staging and output stage where it is large.
//
// Against the any-alignment gather: 7 x 7 stride 2, 3 -> 64 channels on eight images of 224 x 224 30.6 -> 11.1 us, on 32
// images 100 -> 28.8; 1 x 1, 3 -> 64 on 22 images of 163 x 163 65 -> 17.2 (2.2 TB/s of output); 3 x 3, 3 -> 80 on two of
// 128 x 128 16.0 -> 6.5; 55 -> 58 on four of 7 x 7 12.2 -> 7.9.
#pragma once
#include <algorithm>
#include "gemm_ragged.hpp"

namespace ac {

struct ConvImageParams {
  int32_t CP;       // bytes of a pixel in LDS
  int32_t PITCH;    // bytes of a patch row
  int32_t RD;       // dwords of a patch row that are staged
  int32_t NC, RPI, p_row, p_c;  // staging: pieces of 64 dwords to a row; rows to a piece where a row is 32 dwords and less;
                                // from one piece of a wave to its next
  int32_t RUNP;     // K bytes of one kernel row, padded to whole chunks
  int32_t U, units; // units per image, units
  int32_t patch;    // bytes of the patch, slack included
  int32_t rin_max;  // most input rows of a unit
  int32_t w_bytes;  // bytes of the weights
  FastDiv dRD, dCP, dRUNP, dNC;
  unsigned cpd_magic, cpd_one;  // x / (CP / 4)
  unsigned u_magic, ow_magic;  // x / U and x / OW for units and pixels of an image by one multiply; 0: by a division
};

struct __attribute__((packed, aligned(4))) Dwords16 {
  v4i v;
};

template <int BM, int BN>
__global__ void __launch_bounds__(2 * BM) __attribute__((amdgpu_waves_per_eu(4))) conv_i8_image_kernel(const GemmParams p, const ConvImageParams h, const int n_blocks) {
  using T = TypeI8;
  constexpr int THREADS = 2 * BM, WAVES = THREADS / 64, TN = BN / 32, B_STRIDE = BN + 16, CPR = BN / 16, WB = 1024 / THREADS, PB = 8;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int* const bias = (int*)(smem + h.patch);
  unsigned char* const Bs = smem + h.patch + BN * 4;
  const int wgs = gridDim.x / n_blocks, wg = blockIdx.x / n_blocks;
  const int n0 = (blockIdx.x - wg * n_blocks) * BN;
  const int npix = p.OH * p.OW, CPD = h.CP >> 2;
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
  // ---- the input rows of a unit.  A wave takes pieces wave, wave + WAVES, ...: 64 dwords of a row, or RPI short rows;
  // padding pixels are beyond the range of the bounds check and come back as zeros. ----
  const int sub = h.RPI > 1 ? (int)h.dRD.div((unsigned)lane) : 0;
  const int j0 = lane - sub * h.RD;  // dword of the row in piece 0
  const int row_bytes = p.W * p.Cin;
  struct Piece {
    int prow, c;  // piece row (RPI input rows) and piece of it
  };
  auto next_piece = [&](Piece& q) {
    q.prow += h.p_row, q.c += h.p_c;
    if (q.c >= h.NC) q.c -= h.NC, q.prow++;
  };
  int preg[PB];
  auto patch_load = [&](const Unit& w, Piece q) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)p.A, 0, p.a_bytes, 0x00020000);
    const int img = w.img * p.H * row_bytes;  // (an input has fewer than 2^31 bytes)
    int jj = j0, ss = sub;
    asm volatile("" : "+v"(jj), "+v"(ss));  // the positions are computed afresh for every unit: kept, they fill the register file
#pragma unroll
    for (int i = 0; i < PB; i++) {
      if (i % 2 == 0 && q.prow * h.RPI >= w.rin) break;  // (wave-uniform; small patches have one or two pieces to a wave)
      const int j = jj + q.c * 64, px = (int)(__umulhi((unsigned)j, h.cpd_magic) + ((unsigned)j & h.cpd_one)), cd = j - __mul24(px, CPD);
      const int ih = w.ih0 + q.prow * h.RPI + ss, iw = px - p.pad;
      const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
      int off = img + __mul24(ih, row_bytes) + __mul24(iw, p.Cin) + 4 * cd;
      // the last dword of the input may have fewer than 4 bytes behind it
      const int over = off > p.a_bytes - 4 ? off - (p.a_bytes - 4) : 0;
      off = in ? off - over : -1;
      preg[i] = (int)((unsigned)__builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 0) >> (8 * (over & 3)));
      next_piece(q);
    }
  };
  auto patch_store = [&](const Unit& w, Piece q) {
    int jj = j0, ss = sub;
    asm volatile("" : "+v"(jj), "+v"(ss));
    if (ss >= h.RPI) ss = 1 << 20;
#pragma unroll
    for (int i = 0; i < PB; i++) {
      if (i % 2 == 0 && q.prow * h.RPI >= w.rin) break;
      const int row = q.prow * h.RPI + ss, j = jj + q.c * 64;
      if (row < w.rin && j < h.RD) *(int*)(smem + __mul24(row, h.PITCH) + 4 * j) = preg[i];
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
      const int kw = (int)h.dCP.div((unsigned)r), ci = r - kw * h.CP;
      const int col = n0 + cc * 16;
      const bool in = kh < p.KH && kw < p.KW && ci < p.Cin && col < p.N;
      int g = ((kh * p.KW + kw) * p.Cin + ci) * p.N + col;
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
    // this lane's pixel (beyond the image: the last one) and its first patch byte
    const int qi = w.q0 + wave * 32 + (lane & 31);
    const int x = w.ow0 + (qi < npix ? qi : npix - 1) - w.q0;
    const int pr = (int)p.dOW.div((unsigned)x), pc = x - pr * p.OW;
    const int pix = (pr * h.PITCH + pc * h.CP) * p.stride;

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
    auto read = [&](int s) {
      a[s] = ((const Dwords16*)(smem + off))->v;
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

// Geometry for units of bm pixels and column blocks of bn, or false when the convolution does not fit (its input rows
// or the weights of one kernel row are too large for LDS).
static inline bool conv_image_plan(const GemmParams& p, int bm, int bn, ConvImageParams* h, size_t* lds) {
  const int64_t w_bytes = (int64_t)p.K * p.N, npix = (int64_t)p.OH * p.OW;
  if (p.Cin < 1 || p.KH < 1 || p.KW < 1 || npix < 1 || npix >= (1ll << 31) || p.M % npix != 0 || p.a_bytes < 4 || w_bytes < 16 || w_bytes >= (1ll << 31) || p.N >= (1 << 29)) return false;
  if ((p.bias != nullptr && p.bias_ld != 0) || p.shift < 1 || p.shift > 17) return false;  // (the rounding of the other shifts is not built into it)
  const int64_t cp = ((int64_t)p.Cin + 3) / 4 * 4, wp = (int64_t)(p.OW - 1) * p.stride + p.KW;
  const int64_t span = std::min<int64_t>((bm + p.OW - 2) / p.OW + 1, p.OH);  // output rows that bm consecutive pixels can touch
  const int64_t rin = (span - 1) * p.stride + p.KH, pitch = (wp * cp + 15) / 16 * 16, runp = (p.KW * cp + 15) / 16 * 16;
  // one row and one chunk of slack: the reads of the padding of a run, and of an odd last chunk
  const int64_t patch = (rin + 1) * pitch + 32, budget = 160 * 1024;
  if (cp > 4096 || runp > 32768 || pitch > budget || patch > budget - 4096) return false;
  const int64_t need = patch + bn * 4 + (p.KH * runp + 31) / 32 * 32 * (bn + 16);
  if (need > budget) return false;
  const int64_t units_per_image = (npix + bm - 1) / bm, units = p.M / npix * units_per_image;
  if (units > (1 << 30)) return false;
  h->CP = (int32_t)cp, h->PITCH = (int32_t)pitch, h->RD = (int32_t)(wp * cp / 4), h->RUNP = (int32_t)runp;
  h->U = (int32_t)units_per_image, h->units = (int32_t)units, h->patch = (int32_t)patch, h->rin_max = (int32_t)rin, h->w_bytes = (int32_t)w_bytes;
  h->NC = (h->RD + 63) / 64, h->RPI = h->RD <= 32 ? 64 / h->RD : 1;
  h->p_row = bm / 32 / h->NC, h->p_c = bm / 32 - h->p_row * h->NC;
  if (p.H >= (1 << 23) || p.W >= (1 << 23) || (int64_t)p.W * p.Cin >= (1 << 23)) return false;  // 24-bit products
  h->u_magic = units * units_per_image < (1ll << 32) ? FastDiv::make(h->U).magic : 0;
  h->ow_magic = npix * p.OW < (1ll << 32) ? FastDiv::make(p.OW).magic : 0;
  h->dNC = FastDiv::make(h->NC), h->dRD = FastDiv::make(h->RD), h->cpd_magic = FastDiv::make(h->CP / 4).magic, h->cpd_one = h->CP == 4 ? ~0u : 0u, h->dCP = FastDiv::make(h->CP), h->dRUNP = FastDiv::make(h->RUNP);
  *lds = (size_t)need;
  return true;
}

template <int BM, int BN>
static hipError_t launch_conv_image_kernel(const GemmParams& p, const ConvImageParams& h, size_t lds, hipStream_t stream) {
  auto kern = conv_i8_image_kernel<BM, BN>;
  static std::atomic<bool> configured{false};
  if (const hipError_t e = allow_dynamic_lds_once(configured, kern, 160 * 1024)) return e;
  const int n_blocks = (p.N + BN - 1) / BN;
  // workgroups resident on a compute unit: by LDS, and 1024 threads
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(160 * 1024 / (int64_t)lds, 1024 / (2 * BM)));
  int64_t wgs = per_cu * compute_units() / n_blocks;
  if (wgs < 1) wgs = 1;
  if (wgs > h.units) wgs = h.units;
  hipLaunchKernelGGL(kern, dim3((unsigned)(wgs * n_blocks)), dim3(2 * BM), lds, stream, p, h, n_blocks);
  return hipGetLastError();
}

// Launches the kernel when it takes the convolution and is the faster one; false otherwise.
static inline bool launch_conv_image(const GemmParams& p, hipStream_t stream, hipError_t* e) {
  // the block width that computes the fewest columns beyond N
  auto cost = [&](int bn) { return (int64_t)((p.N + bn - 1) / bn) * (bn + 16); };
  const int bn = cost(96) <= cost(64) && cost(96) <= cost(32) ? 96 : (cost(64) <= cost(32) ? 64 : 32);
  ConvImageParams h;
  size_t lds = 0;
  if (!conv_image_plan(p, 128, bn, &h, &lds)) return false;
  // A single tap reuses nothing of the patch and is a plain product, for which the any-alignment GEMM has whole chunks
  // from 64 channels on (eight images of 14 x 14: 60 -> 60 channels 9.6 us there and 6.9 here on 256 images, 130 -> 100
  // 6.1 and 7.9, 512 -> 250 7.4 and 17.9).  From 64 K-steps on the weights of a block are most of the work, and a
  // workgroup has them to itself (51 -> 28 channels, 7 x 7 on three images of 19 x 19, 81 K-steps: 13.7 us cut along K
  // there, 20 here; 40 -> 20, 7 x 7 on eight of 56 x 56, 63 K-steps: 28 and 18).
  if (p.KH * h.RUNP > 64 * 32 || (p.KH * p.KW == 1 && p.Cin > 64)) return false;
  // Units of 256 pixels where 128 would restage the rows under their windows too often (more than 12 dwords a pixel)
  // and 256 still gives every compute unit one: 7 x 7 with stride 2 on eight images of 224 x 224 x 3 11.1 us against
  // 12.3 with 128, 3 x 3 on five of 211 x 211 x 1 13.7 against 11.9.
  const int64_t nblk = (p.N + bn - 1) / bn;
  ConvImageParams h256;
  size_t lds256 = 0;
  const bool big = (int64_t)h.rin_max * h.RD > 12 * 128 && conv_image_plan(p, 256, bn, &h256, &lds256) && h256.units * nblk >= 256;
  if (big) *e = bn == 96 ? launch_conv_image_kernel<256, 96>(p, h256, lds256, stream) : bn == 64 ? launch_conv_image_kernel<256, 64>(p, h256, lds256, stream) : launch_conv_image_kernel<256, 32>(p, h256, lds256, stream);
  else *e = bn == 96 ? launch_conv_image_kernel<128, 96>(p, h, lds, stream) : bn == 64 ? launch_conv_image_kernel<128, 64>(p, h, lds, stream) : launch_conv_image_kernel<128, 32>(p, h, lds, stream);
  return true;
}

}  // namespace ac
