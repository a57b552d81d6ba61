// int8 convolution of images of few channels (the first layer of a network) for gfx950: kernel rows of at most 32 bytes.
//
// The KW * Cin bytes of a kernel row are contiguous under an output pixel, so one or two 16-byte chunks of K are a kernel row, and
// a lane loads the chunks of its pixel from where they lie into the registers that the MFMA reads: a wave's 32 pixels overlap so
// much that its loads are served by the vector L1 (7 x 7 stride 2 over three channels: seven loads of a kilobyte that touch
// 1.5 KB).  No patch in LDS and no barrier but the one behind the weights: what conv_image.hpp does for longer kernel rows is
// most of a short one's time (of its 9.3 us on eight images of 224 x 224, 1.5 went to the addresses of patch and weights, 1.1
// to copying, 2.2 to seven K-steps that read LDS off its chunks).
//
// Padding: rows outside the image are dropped lane by lane, and the bytes of a chunk that hang over the row's left or right
// edge are the same for every kernel row, one mask per tile.  Most tiles touch no edge and skip both (a wave-uniform
// test).  Where a chunk, or the dword behind it that some forms load too, would leave the input itself, at its first and last
// pixels, the tile's chunks are loaded where 16 bytes exist and shifted.
// Bytes behind a run meet weight rows of zeros.
//
// A wave takes tiles of 32 consecutive pixels, a run of them per XCD, whose L2 then holds its part of the image; the next
// tile's loads are under way while the current one leaves.
//
// Bound: latency on small outputs (weights, barrier, K loop, output stage: 3.3 us where conv_image.hpp took 4.0), instruction
// issue on larger ones (some 100 to 250 a tile), the output's bytes beyond 30 MB.  Against conv_image.hpp on 4000 random such
// convolutions 1.27 in the mean, worst 0.90 (an image of 3 x 5); us before and after: 7 x 7 stride 2, 3 -> 64 on eight images of
// 224 x 224 10.2 / 7.3, on 32 23.4 / 15.3; 3 x 3, 4 -> 16 on 20 of 228 x 228 18.6 / 11.9; 5 x 5, 3 -> 32 on eight of 197 x 197
// 11.1 / 7.1; 1 x 1, 3 -> 64 on ten of 200 x 200 12.4 / 9.5; 3 x 3, 3 -> 16 on one of 32 x 32 4.0 / 3.2.  With loads from any byte the
// first of them 8.5.
#include "conv_direct_rules.hpp"
#include "gemm_ragged.hpp"

namespace ac {

constexpr int CONV_DIRECT_WAVES = 4;

struct ConvDirectArgs {
  const void *A, *B;
  void* C;
  const int32_t* bias;
  int32_t M, N, a_bytes, w_bytes;
  int32_t tiles, per_xcd;  // of 32 pixels; a run of so many to an XCD, 0: dealt over the workgroups in turn
  int32_t Cin, stride;
  uint16_t H, W, OH, OW, KH, RUN, pad;
  uint8_t shift, act;
  FastDiv dOW, dOH;
};
static_assert(sizeof(ConvDirectArgs) <= 112, "beyond, a launch costs more");

// NKS: K-steps of 32 bytes.  NARROW: a kernel row is one chunk, two rows to a K-step; otherwise two chunks.
template <int NKS, int TN, bool NARROW, ConvDirectShift SHIFT>
__global__ void __launch_bounds__(64 * CONV_DIRECT_WAVES) __attribute__((amdgpu_waves_per_eu(TN == 3 ? 3 : 4))) conv_i8_direct_kernel(const ConvDirectArgs p) {
  using T = TypeI8;
  constexpr int WAVES = CONV_DIRECT_WAVES, BN = 32 * TN, B_STRIDE = BN + 16, CPR = BN / 16, THREADS = 64 * WAVES, NROW = 32 * NKS, PAYLOAD = conv_direct_payload(SHIFT);
  constexpr int WB = (NROW * CPR + THREADS - 1) / THREADS;  // chunks of the weights per thread
  constexpr bool RESIDENT = NKS * TN <= 6;                  // the weights' fragments stay in registers
  __shared__ __attribute__((aligned(16))) int bias[BN];
  __shared__ __attribute__((aligned(16))) unsigned char Bs[NROW * B_STRIDE];
  const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n0 = blockIdx.y * BN, xcd = blockIdx.x & 7;
  const int row_bytes = p.W * p.Cin;
  const unsigned char* const image = (const unsigned char*)p.A;

  const bool apart = p.per_xcd > 0;
  int tile = apart ? xcd * p.per_xcd + (int)(blockIdx.x >> 3) * WAVES : (int)blockIdx.x * WAVES;
  const int tile_end = apart && (xcd + 1) * p.per_xcd < p.tiles ? (xcd + 1) * p.per_xcd : p.tiles, tile_step = (int)(apart ? gridDim.x >> 3 : gridDim.x) * WAVES;
  if (tile >= tile_end) return;  // the whole workgroup
  tile += wave;

  // ---- one tile's pixels: position, what of its chunks lies in the image, and the loads ----
  constexpr int READ = conv_direct_read(SHIFT);
  v4i a[NKS];
  int tail[SHIFT == DIRECT_TAIL ? NKS : 1];
  int m, ih0;   // the lane's pixel and the first image row under it
  int base;     // byte of its chunk in kernel row 0
  int lo, hi;   // bytes of its chunks inside an image row, [lo, hi)
  bool whole;   // wave-uniform: no lane's chunks leave the image
  bool near;    // wave-uniform: some would leave the input itself
  auto within = [&](int g) { return g < 0 ? 0 : g > p.a_bytes - 16 ? p.a_bytes - 16 : g; };
  auto request = [&](int tl) {
    m = tl * 32 + (lane & 31);
    const unsigned mm = (unsigned)(m < p.M ? m : p.M - 1);
    const unsigned q = p.dOW.div(mm), img = p.dOH.div(q);
    const int ow = (int)(mm - q * p.OW), oh = (int)(q - img * p.OH);
    ih0 = oh * p.stride - p.pad;
    const int col = (ow * p.stride - p.pad) * p.Cin, b = col + (NARROW ? 0 : PAYLOAD * half);
    base = ((int)img * p.H + ih0) * row_bytes + b;
    const ConvDirectWindow window = {ih0, col, base};
    whole = __all(conv_direct_whole(window, p.H, p.KH, p.RUN, row_bytes, p.a_bytes, READ));
    auto row_of = [&](int ks) { return NARROW ? 2 * ks + half : ks; };
    auto load = [&](int ks, int g) {
      if constexpr (SHIFT != DIRECT_NONE) g &= ~3;
      a[ks] = ((const Dwords16*)(image + (unsigned)g))->v;
      if constexpr (SHIFT == DIRECT_TAIL) tail[ks] = *(const int*)(image + (unsigned)g + 16);
    };
    if (whole) {
#pragma unroll
      for (int ks = 0; ks < NKS; ks++) {
        int kh = row_of(ks);
        if (NARROW && ks == NKS - 1) kh = kh < p.KH ? kh : p.KH - 1;  // an odd number of rows
        load(ks, base + kh * row_bytes);
      }
    } else {
      lo = b < 0 ? -b : 0, hi = row_bytes - b;
      hi = hi < 0 ? 0 : hi > 16 ? 16 : hi;  // (a chunk's bytes beyond its payload meet zeros)
      lo = lo > 16 ? 16 : lo;
      const int first = ih0 < 0 ? -ih0 : 0, last = p.H - 1 - ih0 < p.KH - 1 ? p.H - 1 - ih0 : p.KH - 1;  // kernel rows inside the image
      near = !__all(conv_direct_fits(window, first, last, row_bytes, p.a_bytes, READ));
#pragma unroll
      for (int ks = 0; ks < NKS; ks++) {
        const int kh = row_of(ks);
        const int g = (kh >= first) & (kh <= last) ? base + kh * row_bytes : 0;
        if (near) a[ks] = load16_any(image + (unsigned)within(g));
        else load(ks, g);
      }
    }
  };
  // chunks to their first byte
  auto align = [&] {
#pragma unroll
    for (int ks = 0; ks < NKS; ks++) {
      int kh = NARROW ? 2 * ks + half : ks;
      if (NARROW && ks == NKS - 1) kh = kh < p.KH ? kh : p.KH - 1;
      const unsigned s = (unsigned)(base + kh * row_bytes) & 3u;
      const v4i w = a[ks];
#pragma unroll
      for (int e = 0; e < 4; e++) a[ks][e] = (int)__builtin_amdgcn_alignbyte((unsigned)(e < 3 ? w[e + 1] : SHIFT == DIRECT_TAIL ? tail[ks] : 0), (unsigned)w[e], s);
    }
  };
  // rows and bytes outside the image to zeros
  auto cut = [&] {
    if (near) {  // a row at an end of the input, of the pixels at an edge of it
#pragma unroll
      for (int ks = 0; ks < NKS; ks++) {
        const int g = base + (NARROW ? 2 * ks + half : ks) * row_bytes, s = g - within(g);
        a[ks] = chunk_apply<true>(a[ks], (s < -16) | (s > 16) ? chunk_fix(0, 0, 0) : chunk_fix(s, 0, 16));
      }
    }
    Chunk c = chunk_down({~(uint64_t)0, ~(uint64_t)0}, 16 - hi);
    const Chunk l = chunk_up({~(uint64_t)0, ~(uint64_t)0}, lo);
    c.a &= l.a, c.b &= l.b;
    const int mask[4] = {(int)(unsigned)c.a, (int)(unsigned)(c.a >> 32), (int)(unsigned)c.b, (int)(unsigned)(c.b >> 32)};
#pragma unroll
    for (int ks = 0; ks < NKS; ks++) {
      const int ih = ih0 + (NARROW ? 2 * ks + half : ks);
      const bool in = (unsigned)ih < (unsigned)p.H;
#pragma unroll
      for (int d = 0; d < 4; d++) a[ks][d] = in ? a[ks][d] & mask[d] : 0;
    }
  };

  // ---- weights: kernel rows of RUN bytes of K padded to RUNP, requested together with the first tile ----
  v4i wreg[WB];
  int wpos[WB];  // byte of the weights; beyond the last 16 of them, where a chunk is loaded early
#pragma unroll
  for (int i = 0; i < WB; i++) {
    const int idx = i * THREADS + t, k = idx / CPR, c = n0 + (idx - k * CPR) * 16;
    const int kh = NARROW ? k / 16 : k / 32, r = NARROW ? k % 16 : k % 16 + PAYLOAD * (k / 16 % 2);
    wpos[i] = (kh < p.KH) & (k % 16 < PAYLOAD) & (r < p.RUN) & (c < p.N) ? (kh * p.RUN + r) * p.N + c : -1;
    const int q = wpos[i] < 0 ? 0 : wpos[i] < p.w_bytes - 16 ? wpos[i] : p.w_bytes - 16;
    wreg[i] = load16_any((const unsigned char*)p.B + (unsigned)q);
  }
  const int my_bias = p.bias && t < BN && n0 + t < p.N ? p.bias[n0 + t] : 0;
  if (tile < tile_end) request(tile);
#pragma unroll
  for (int i = 0; i < WB; i++) {
    const int idx = i * THREADS + t, k = idx / CPR;
    v4i v = wreg[i];
    if (p.N % 16 != 0 && wpos[i] > p.w_bytes - 16) v = chunk_apply<false>(v, chunk_fix(wpos[i] - (p.w_bytes - 16), 0, 16));
#pragma unroll
    for (int e = 0; e < 4; e++) v[e] = wpos[i] < 0 ? 0 : v[e];
    if (NROW * CPR % THREADS == 0 || k < NROW) *(v4i*)(Bs + k * B_STRIDE + (idx - k * CPR) * 16) = v;
  }
  if (t < BN) bias[t] = my_bias;
  block_sync();

  const unsigned char* const bp = Bs + (half * 16 + ((lane & 15) >> 1)) * B_STRIDE + 16 * ((lane >> 4) & 1) + 8 * (lane & 1);
  auto column = [&](int ks, int j) {
    const v2i l = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, bp + 32 * ks * B_STRIDE + 32 * j));
    const v2i h = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, bp + (32 * ks + 8) * B_STRIDE + 32 * j));
    return (v4i){l[0], l[1], h[0], h[1]};
  };
  v4i fixed[RESIDENT ? NKS : 1][TN];
  if constexpr (RESIDENT) {
#pragma unroll
    for (int ks = 0; ks < NKS; ks++)
#pragma unroll
      for (int j = 0; j < TN; j++) fixed[ks][j] = column(ks, j);
  }
  const EpilogueI8::FastQuant f = EpilogueI8::fast_quant(p.shift, p.act);
#pragma unroll 1
  while (tile < tile_end) {
    typename T::accv acc[TN];
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const v4i b4 = *(const v4i*)(bias + 32 * j + 8 * q + 4 * half);
#pragma unroll
        for (int e = 0; e < 4; e++) acc[j][4 * q + e] = b4[e];
      }
    if constexpr (SHIFT != DIRECT_NONE)
      if (whole || !near) align();
    if (!whole) cut();
#pragma unroll
    for (int ks = 0; ks < NKS; ks++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[j] = T::mfma(RESIDENT ? fixed[ks][j] : column(ks, j), a[ks], acc[j]);
    const int pixel = m;
    if ((tile += tile_step) < tile_end) request(tile);

    // ---- output stage: a lane holds 16 consecutive columns of its pixel after the exchange ----
    int8_t* const row = (int8_t*)p.C + (int64_t)pixel * p.N;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      if (n0 + 32 * j >= p.N) break;
      int v[16];
#pragma unroll
      for (int e = 0; e < 16; e++) v[e] = acc[j][e];
      const v4i o = EpilogueI8::quant16<true>(v, f);
      const int n = n0 + 32 * j + 16 * half;
      if (pixel < p.M) store_run16(row + n, o, p.N - n);
      __builtin_amdgcn_sched_barrier(0);  // one column tile at a time: interleaved, the values of all of them spill
    }
  }
}

template <int NKS, int TN, bool NARROW, ConvDirectShift SHIFT>
static hipError_t launch_conv_direct_cfg(ConvDirectArgs& a, int n_blocks, hipStream_t stream) {
  constexpr int WAVES = CONV_DIRECT_WAVES;
  const int64_t wgs = (((int64_t)a.tiles + 7) / 8 + WAVES - 1) / WAVES * 8, most = (int64_t)compute_units() * ((TN == 3 ? 12 : 16) / WAVES) / n_blocks / 8 * 8;
  const int64_t grid = wgs < most ? wgs : most < 8 ? 8 : most;
  return launch_kernel(conv_i8_direct_kernel<NKS, TN, NARROW, SHIFT>, dim3((unsigned)grid, (unsigned)n_blocks), dim3(64 * WAVES), 0, stream, a);
}
template <int TN, bool NARROW, ConvDirectShift SHIFT>
static hipError_t launch_conv_direct_steps(int nks, ConvDirectArgs& a, int n_blocks, hipStream_t stream) {
  switch (nks) {
    case 1: return launch_conv_direct_cfg<1, TN, NARROW, SHIFT>(a, n_blocks, stream);
    case 2: return launch_conv_direct_cfg<2, TN, NARROW, SHIFT>(a, n_blocks, stream);
    case 3: return launch_conv_direct_cfg<3, TN, NARROW, SHIFT>(a, n_blocks, stream);
    case 4: return launch_conv_direct_cfg<4, TN, NARROW, SHIFT>(a, n_blocks, stream);
  }
  if constexpr (!NARROW) {
    switch (nks) {
      case 5: return launch_conv_direct_cfg<5, TN, NARROW, SHIFT>(a, n_blocks, stream);
      case 6: return launch_conv_direct_cfg<6, TN, NARROW, SHIFT>(a, n_blocks, stream);
      case 7: return launch_conv_direct_cfg<7, TN, NARROW, SHIFT>(a, n_blocks, stream);
    }
  }
  return hipErrorInvalidValue;
}
template <bool NARROW, ConvDirectShift SHIFT>
static hipError_t launch_conv_direct_columns(int bn, int nks, ConvDirectArgs& a, int n_blocks, hipStream_t stream) {
  return bn == 96 ? launch_conv_direct_steps<3, NARROW, SHIFT>(nks, a, n_blocks, stream)
       : bn == 64 ? launch_conv_direct_steps<2, NARROW, SHIFT>(nks, a, n_blocks, stream) : launch_conv_direct_steps<1, NARROW, SHIFT>(nks, a, n_blocks, stream);
}
template <bool NARROW>
static hipError_t launch_conv_direct_shift(ConvDirectShift shift, int bn, int nks, ConvDirectArgs& a, int n_blocks, hipStream_t stream) {
  return shift == DIRECT_NONE ? launch_conv_direct_columns<NARROW, DIRECT_NONE>(bn, nks, a, n_blocks, stream)
       : shift == DIRECT_13 ? launch_conv_direct_columns<NARROW, DIRECT_13>(bn, nks, a, n_blocks, stream) : launch_conv_direct_columns<NARROW, DIRECT_TAIL>(bn, nks, a, n_blocks, stream);
}

// Launches the kernel when it takes the convolution; false otherwise.
bool launch_conv_direct(const GemmParams& p, hipStream_t stream, hipError_t* e) {
  if (p.bias != nullptr && p.bias_ld != 0) return false;
  const ConvDirectForm f = conv_direct_form({p.M, p.N, p.K, p.H, p.W, p.Cin, p.KH, p.KW, p.OH, p.OW, p.stride, p.pad, p.a_bytes, p.shift, ((uintptr_t)p.A & 3) == 0});
  if (!f.takes) return false;
  ConvDirectArgs a = {};
  a.A = p.A, a.B = p.B, a.C = p.C, a.bias = p.bias;
  a.M = p.M, a.N = p.N, a.a_bytes = p.a_bytes, a.w_bytes = p.K * p.N;
  a.tiles = (int32_t)(((int64_t)p.M + 31) / 32), a.per_xcd = (int64_t)p.M * p.N <= 32 << 20 ? (a.tiles + 7) / 8 : 0;
  a.Cin = p.Cin, a.stride = p.stride;
  a.H = (uint16_t)p.H, a.W = (uint16_t)p.W, a.OH = (uint16_t)p.OH, a.OW = (uint16_t)p.OW, a.KH = (uint16_t)p.KH, a.RUN = (uint16_t)(p.KW * p.Cin), a.pad = (uint16_t)p.pad;
  a.shift = (uint8_t)p.shift, a.act = (uint8_t)p.act;
  a.dOW = p.dOW, a.dOH = p.dOH;
  *e = f.narrow ? launch_conv_direct_shift<true>(f.shift, f.bn, f.nks, a, (int)f.n_blocks, stream) : launch_conv_direct_shift<false>(f.shift, f.bn, f.nks, a, (int)f.n_blocks, stream);
  return true;
}

}  // namespace ac
