// GEMM and convolution with few output tiles and a deep K: the waves of a workgroup share one 32 x 32 tile of C and
// take its K tiles in turn.
//
// With fewer tiles than compute units a launch lasts as long as one tile's K loop, and one wave (or four waves on a
// 64 x 64 tile) has too few loads in flight to stream its operands: the loop is a chain of latencies.  Cutting K over
// workgroups fixes that and costs a second launch and a workspace, which half of the entry points do not have.  Here the
// cut stays inside the workgroup: wave w of W multiplies K tiles w, w + W, ... out of LDS of its own (no barrier in the
// loop), then every wave leaves its accumulators in LDS, four waves sum them in wave order (the same bits on every run)
// and run the output stage.  Two kernels: aligned operands stream through direct-to-LDS rings (gemm_dtl.hpp), any others
// through registers (gemm_ragged.hpp).
#pragma once
#include "gemm_ragged.hpp"
#include "gemm_rules.hpp"

namespace ac {

// Output stages of four columns n .. n + 3 of row m, or of those of them that exist.  `bias` is what prefetch() returned.
struct KGroupBias {
  template <class P>
  static __device__ __forceinline__ v4i prefetch(const P& p, int m, int n) {
    v4i b = {0, 0, 0, 0};
    if (p.bias != nullptr) {
      const int32_t* row = p.bias + (int64_t)m * p.bias_ld + n;  // bias_ld 0: one row for all
      if (n + 3 < p.N) {
        b = ((const Unaligned16*)row)->v;
      } else {
#pragma unroll
        for (int e = 0; e < 3; e++) b[e] = row[n + e < p.N ? e : 0];
      }
    }
    return b;
  }
};
struct KGroupI8 : KGroupBias {
  typedef int val;
  template <class P>
  static __device__ __forceinline__ void store(const P& p, int m, int n, v4i s, v4i bias) {
    s += bias;
    int q[4];
    if (p.shift >= 1 && p.shift <= 23) {
      const EpilogueI8::FastQuant f = EpilogueI8::fast_quant(p.shift, p.act);
#pragma unroll
      for (int e = 0; e < 4; e++) q[e] = p.shift <= 17 ? EpilogueI8::requant_fast<true>(s[e], f) : EpilogueI8::requant_fast<false>(s[e], f);
    } else {
#pragma unroll
      for (int e = 0; e < 4; e++) q[e] = EpilogueI8::requant(s[e], p.shift, p.act);
    }
    struct __attribute__((packed)) U4 { unsigned v; };
    int8_t* dst = (int8_t*)p.C + (int64_t)m * p.ldc + n;
    if (n + 3 < p.N) {
      ((U4*)dst)->v = EpilogueI8::pack4(q[0], q[1], q[2], q[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 3; e++)
        if (n + e < p.N) dst[e] = (int8_t)q[e];
    }
  }
};
struct KGroupRawI32 : KGroupBias {
  typedef int val;
  template <class P>
  static __device__ __forceinline__ void store(const P& p, int m, int n, v4i s, v4i bias) {
    s += bias;
    int32_t* dst = (int32_t*)p.C + (int64_t)m * p.ldc + n;
    if (n + 3 < p.N) {
      ((Unaligned16*)dst)->v = s;
    } else {
#pragma unroll
      for (int e = 0; e < 3; e++)
        if (n + e < p.N) dst[e] = s[e];
    }
  }
};
struct KGroupF32 {
  typedef float val;
  template <class P>
  static __device__ __forceinline__ v4i prefetch(const P&, int, int) { return (v4i){0, 0, 0, 0}; }
  template <class P>
  static __device__ __forceinline__ void store(const P& p, int m, int n, v4f s, v4i) {
    struct __attribute__((packed)) U16 { v4f v; };
    float* dst = (float*)p.C + (int64_t)m * p.ldc + n;
    if (n + 3 < p.N) {
      v4f o = p.alpha * s;
      if (p.beta != 0.f) o += p.beta * ((const U16*)dst)->v;
      ((U16*)dst)->v = o;
    } else {
#pragma unroll
      for (int e = 0; e < 3; e++)
        if (n + e < p.N) EpilogueF32::one(p, m, n + e, s[e]);
    }
  }
};

// The waves' sums of a 32 x 32 tile (swapped operand order: a lane holds runs of four columns of its row) meet in LDS, one
// region of 4 KB per wave, PITCH bytes apart: columns 4 c .. 4 c + 3 of row r in slot r ^ c of group c, so that the eight
// threads of a row read different banks.  Threads 0 .. 255 sum them and own row t / 8, columns 4 (t % 8) + 0 .. 3.
template <class OUT, int W, int PITCH, class ACC, class P>
static __device__ __forceinline__ void kgroup_finish(const P& p, unsigned char* smem, int wave, int t, const ACC& acc, int om, int on, bool out, v4i bias) {
  typedef typename OUT::val val;
  typedef val v4 __attribute__((ext_vector_type(4)));
  const int lane = t & 63;
#pragma unroll
  for (int g = 0; g < 4; g++) {
    const int c = 2 * g + (lane >> 5), r = lane & 31;
    *(v4*)(smem + wave * PITCH + c * 512 + ((r ^ c) << 4)) = (v4){acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
  }
  block_sync();
  if (!out) return;
  const int c = t & 7, r = t >> 3;
  const unsigned char* src = smem + c * 512 + ((r ^ c) << 4);
  v4 s = *(const v4*)src;
#pragma unroll
  for (int w = 1; w < W; w++) s += *(const v4*)(src + w * PITCH);
  OUT::store(p, om, on, s, bias);
}

// KTB: bytes of K per tile, S: stages of a wave's ring, W: waves of a workgroup; AMODE, TA, TB, DW as for gemm_dtl_kernel.
template <class T, class OUT, int KTB, int S, int W, int AMODE, bool TA, bool TB, bool DW>
__global__ void __launch_bounds__(64 * W) gemm_kgroup_kernel(const std::conditional_t<AMODE == 1, ConvArgs, GemmArgs> p) {
  using G = DtlGeometry<T, 32, 32, 1, 1, S, KTB>;
  constexpr int EB = T::EB, NA = G::A_INSTR, NB = G::B_INSTR, KS = G::KSTEPS, PER_TILE = NA + NB;
  static_assert(G::STAGE == 64 * KTB && S >= 3 && S * G::STAGE >= 4096 && W >= 4, "geometry");
  static_assert((S - 1) * PER_TILE <= 63, "vmcnt is a 6-bit counter");
  static_assert(!(TA || TB) || (AMODE == 0 && EB == 1), "transposed operands: int8 GEMM");
  constexpr int AT_ROW = G::B_ROW, AT_SPR = G::B_SPR, AT_RPI = G::B_ROWS_PER_INSTR;  // A^T takes B's form in LDS
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  unsigned char* win = smem + wave * (S * G::STAGE);
  const unsigned lds0 = (unsigned)(uintptr_t)AC_LDS(unsigned char, win);
  const int tiles_m = (p.M + 31) / 32, tiles_n = (p.N + 31) / 32;
  int tm, tn;
  tile_coords_mul(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, p.band_magic, tm, tn);
  const int m0 = tm * 32, n0 = tn * 32;
  const int kbytes = p.K * EB;
  const unsigned char* zero = (const unsigned char*)g_zero16;

  // outputs of this thread in the end (threads 0 .. 255); the bias is requested ahead of the operands
  const int om = m0 + (t >> 3), on = n0 + 4 * (t & 7);
  const bool out = t < 256 && om < p.M && on < p.N;
  v4i bias = {0, 0, 0, 0};
  if (out) bias = OUT::prefetch(p, om, on);

  // source offsets of the loads of a K tile (lane roles of gemm_dtl_kernel, with one wave)
  constexpr int NVAR = KTB == 128 ? 2 : 1;
  int a_chunk[NVAR];
#pragma unroll
  for (int v = 0; v < NVAR; v++) a_chunk[v] = (lane % G::A_SPR) ^ G::a_xor(v * G::A_ROWS_PER_INSTR + lane / G::A_SPR);
  unsigned a_voff[NA], b_voff[NB];
  int g_base[NA];
  unsigned g_rows[NA], g_cols[NA], g_kb[NVAR];
  v4i a_rsrc = {0, 0, 0, 0};
  if constexpr (AMODE == 1) {
    const uint64_t ab = (uint64_t)(uintptr_t)p.A;
    a_rsrc[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)ab);
    a_rsrc[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(ab >> 32));
    a_rsrc[2] = __builtin_amdgcn_readfirstlane(p.a_bytes);
    a_rsrc[3] = 0x00020000;
#pragma unroll
    for (int v = 0; v < NVAR; v++) g_kb[v] = (unsigned)(wave * KTB + a_chunk[v] * 16);
  }
#pragma unroll
  for (int i = 0; i < NA; i++) {
    const int row = i * G::A_ROWS_PER_INSTR + lane / G::A_SPR;
    g_base[i] = 0, g_rows[i] = g_cols[i] = 0u, a_voff[i] = 0u;
    if constexpr (TA) {
      a_voff[i] = (unsigned)(i * AT_RPI + lane / AT_SPR) * (unsigned)p.lda + (m0 + (lane % AT_SPR) * 16 < p.M ? (lane % AT_SPR) * 16 : 0);
    } else if constexpr (AMODE == 0) {
      a_voff[i] = (unsigned)(m0 + row < p.M ? row : p.M - 1 - m0) * (unsigned)(p.lda * EB) + a_chunk[i & (NVAR - 1)] * 16;
    } else {
      const int m = m0 + row;
      const unsigned mm = m < p.M ? (unsigned)m : 0u;
      const unsigned q = p.dOW.div(mm), img = p.dOH.div(q);
      const int ow = (int)(mm - q * p.OW), oh = (int)(q - img * p.OH);
      const int ih0 = oh * p.stride - p.pad, iw0 = ow * p.stride - p.pad;
      g_base[i] = (((int)img * p.H + ih0) * p.W + iw0) * p.Cin;
      g_rows[i] = m < p.M ? span_bits(ih0, p.KH, p.H) : 0u;
      g_cols[i] = span_bits(iw0, p.KW, p.W);
    }
  }
#pragma unroll
  for (int i = 0; i < NB; i++) {
    if constexpr (TB) {
      const int row = i * G::A_ROWS_PER_INSTR + lane / G::A_SPR;
      b_voff[i] = (unsigned)(n0 + row < p.N ? row : p.N - 1 - n0) * (unsigned)p.ldb + a_chunk[i & (NVAR - 1)] * 16;
    } else {
      const int col = (lane % G::B_SPR) * 16;
      b_voff[i] = (unsigned)(i * G::B_ROWS_PER_INSTR + lane / G::B_SPR) * (unsigned)(p.ldb * EB) + (n0 * EB + col < p.N * EB ? col : 0);
    }
  }
  const int64_t a_step = TA ? (int64_t)G::BK * p.lda : (int64_t)KTB, b_step = TB ? (int64_t)KTB : (int64_t)G::BK * p.ldb * EB;
  const unsigned char* a_base = (const unsigned char*)p.A + (TA ? (int64_t)m0 : AMODE == 0 ? (int64_t)m0 * p.lda * EB : 0) + wave * a_step;
  const unsigned char* b_base = (const unsigned char*)p.B + (TB ? (int64_t)n0 * p.ldb : (int64_t)n0 * EB) + wave * b_step;
  const int nkt_total = (kbytes + KTB - 1) / KTB;
  const int nkt = nkt_total > wave ? (nkt_total - wave + W - 1) / W : 0;

  int wr = 0, kt_issue = wave;  // stage and K tile of the next request
  auto issue = [&]() __attribute__((always_inline)) {
    const unsigned st = lds0 + wr * G::STAGE;
    const bool full = (kt_issue + 1) * KTB <= kbytes - (DW ? 1 : 0);  // wave-uniform
    const int kbase = kt_issue * KTB;
    if constexpr (DW) {
      if (!full) {  // the last tile
        const v4i a_tile = buffer_of(a_base, DW_REACH), b_tile = buffer_of(b_base, DW_REACH);
        const int krows = p.K - kbase / EB;  // k-rows left
#pragma unroll
        for (int i = 0; i < NA; i++) {
          if constexpr (TA) {
            dw_load(a_tile, krows - 1, i * AT_RPI, AT_RPI, p.M, i * AT_RPI + lane / AT_SPR < krows ? a_voff[i] : DW_NOTHING, st + i * 1024, lane,
                    [&](int q, int dw) { return dword_strided<EB, AT_ROW>(i * AT_RPI, q, dw, krows, p.M - m0, p.lda); });
          } else {
            dw_load(a_tile, p.M - 1 - m0, i * G::A_ROWS_PER_INSTR, G::A_ROWS_PER_INSTR, kbytes,
                    (i * G::A_ROWS_PER_INSTR + lane / G::A_SPR < p.M - m0) & (kbase + a_chunk[i & (NVAR - 1)] * 16 < kbytes) ? a_voff[i] : DW_NOTHING, st + i * 1024, lane,
                    [&](int q, int dw) { return dword_contiguous<KTB>(i * G::A_ROWS_PER_INSTR, q, dw, p.M - m0, kbytes - kbase, p.lda * EB); });
          }
        }
#pragma unroll
        for (int i = 0; i < NB; i++) {
          const unsigned to = st + G::A_BYTES + i * 1024;
          if constexpr (TB) {
            dw_load(b_tile, p.N - 1 - n0, i * G::A_ROWS_PER_INSTR, G::A_ROWS_PER_INSTR, kbytes,
                    (i * G::A_ROWS_PER_INSTR + lane / G::A_SPR < p.N - n0) & (kbase + a_chunk[i & (NVAR - 1)] * 16 < kbytes) ? b_voff[i] : DW_NOTHING, to, lane,
                    [&](int q, int dw) { return dword_contiguous<KTB>(i * G::A_ROWS_PER_INSTR, q, dw, p.N - n0, kbytes - kbase, p.ldb); });
          } else {
            dw_load(b_tile, krows - 1, i * G::B_ROWS_PER_INSTR, G::B_ROWS_PER_INSTR, p.N * EB,
                    i * G::B_ROWS_PER_INSTR + lane / G::B_SPR < krows ? b_voff[i] : DW_NOTHING, to, lane,
                    [&](int q, int dw) { return dword_strided<EB, G::B_ROW>(i * G::B_ROWS_PER_INSTR, q, dw, krows, (p.N - n0) * EB, p.ldb * EB); });
          }
        }
        wr = wr + 1 == S ? 0 : wr + 1;
        return;
      }
    }
    if constexpr (AMODE == 1) {
      unsigned g_off[NVAR], g_kh[NVAR], g_kw[NVAR], g_dead[NVAR];
#pragma unroll
      for (int v = 0; v < NVAR; v++) {
        const unsigned tap = p.dCin.div(g_kb[v]), ci = g_kb[v] - tap * p.Cin;
        const unsigned kh = p.dKW.div(tap), kw = tap - kh * p.KW;
        g_off[v] = (kh * p.W + kw) * p.Cin + ci;
        g_kh[v] = kh & 31u, g_kw[v] = kw & 31u;
        g_dead[v] = g_kb[v] < (unsigned)kbytes ? 0u : ~0u;
        g_kb[v] += W * KTB;
      }
#pragma unroll
      for (int i = 0; i < NA; i++) {
        const int v = i & (NVAR - 1);
        const unsigned inside = (g_rows[i] >> g_kh[v]) & (g_cols[i] >> g_kw[v]) & 1u;
        buffer_to_lds16(a_rsrc, ((unsigned)g_base[i] + g_off[v]) | (inside - 1u) | g_dead[v], st + i * 1024);
      }
    } else if (full) {
#pragma unroll
      for (int i = 0; i < NA; i++) load_to_lds16_so(a_base, a_voff[i], st + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < NA; i++) {
        const int kb = kbase + (TA ? i * AT_RPI + lane / AT_SPR : a_chunk[i & (NVAR - 1)] * 16);
        load_to_lds16(kb < kbytes ? a_base + a_voff[i] : zero, st + i * 1024);
      }
    }
    if (full) {
#pragma unroll
      for (int i = 0; i < NB; i++) load_to_lds16_so(b_base, b_voff[i], st + G::A_BYTES + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < NB; i++) {
        const int kb = kbase + (TB ? a_chunk[i & (NVAR - 1)] * 16 : (i * G::B_ROWS_PER_INSTR + lane / G::B_SPR) * EB);
        load_to_lds16(kb < kbytes ? b_base + b_voff[i] : zero, st + G::A_BYTES + i * 1024);
      }
    }
    a_base += W * a_step;
    b_base += W * b_step;
    kt_issue += W;
    wr = wr + 1 == S ? 0 : wr + 1;
  };
#pragma unroll
  for (int s = 0; s < S - 1; s++)
    if (s < nkt) issue();

  const int row_off = (lane & 31) * KTB, swz = G::a_xor(lane & 31);  // a K-contiguous fragment: row lane % 32, chunk 2 ks + lane / 32
  const int col_off = dtl_col_off<T, G::B_ROW>((lane >> 5) * 16, 0, lane);
  struct Frag {
    v4i a[KS], b[KS];
  };
  int rd = 0;  // stage of the next tile to be read
  auto read_frags = [&](Frag& f) {
    const unsigned char *As = win + rd * G::STAGE, *Bs = As + G::A_BYTES;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      const int chunk = row_off + (((2 * ks + (lane >> 5)) ^ swz) << 4);
      if constexpr (TA) f.a[ks] = dtl_read_col_at<T, AT_ROW>(As + col_off + ks * (32 / EB) * AT_ROW);
      else f.a[ks] = *(const v4i*)(As + chunk);
      if constexpr (TB) f.b[ks] = *(const v4i*)(Bs + chunk);
      else f.b[ks] = dtl_read_col_at<T, G::B_ROW>(Bs + col_off + ks * (32 / EB) * G::B_ROW);
    }
    rd = rd + 1 == S ? 0 : rd + 1;
  };

  typename T::accv acc = T::zero();
  Frag f[2];
  if (nkt > 0) {
    if (S - 1 <= nkt) wait_vm<(S - 2) * PER_TILE>();
    else wait_vm<0>();
    read_frags(f[0]);
  }
  // As in gemm_i8_small_kernel: request tile kt + S - 1 into the stage that tile kt - 1 has left, wait for this wave's loads
  // of tile kt + 1, read its fragments, then the MFMAs of tile kt.
  auto step = [&](int kt, Frag& cur, Frag& nxt) {
    if (kt + 1 < nkt) {
      if (kt + S - 1 < nkt) {
        issue();
        wait_vm<(S - 2) * PER_TILE>();
      } else {
        wait_vm<0>();
      }
      read_frags(nxt);
    }
    if constexpr (DW && !TA && (TB || EB == 2)) {
      if (kbytes % 16 != 0 && wave + kt * W == nkt_total - 1) {
#pragma unroll
        for (int ks = 0; ks < KS; ks++) cur.a[ks] = dw_mask(cur.a[ks], kbytes - (nkt_total - 1) * KTB - (2 * ks + (lane >> 5)) * 16);
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ks++) acc = T::mfma(cur.b[ks], cur.a[ks], acc);  // swapped: a lane holds runs of four columns of a row
  };
  int kt = 0;
  for (; kt + 1 < nkt; kt += 2) {
    step(kt, f[0], f[1]);
    step(kt + 1, f[1], f[0]);
  }
  if (kt < nkt) step(kt, f[0], f[1]);

  // everything this wave requested has landed and has been read: its sums go where its ring was
  kgroup_finish<OUT, W, S * G::STAGE>(p, smem, wave, t, acc, om, on, out, bias);
}

static inline int64_t kgroup_tiles(const GemmParams& p) { return (int64_t)((p.M + 31) / 32) * ((p.N + 31) / 32); }

template <class ARGS, class T, class KERN>
static hipError_t launch_kgroup_grid(std::atomic<bool>& configured, KERN kern, int waves, int lds, const GemmParams& p, hipStream_t stream) {
  if (const hipError_t e = allow_dynamic_lds_once(configured, kern, lds)) return e;
  const ARGS args = kernel_args<ARGS, T>(p, band_magic_of((p.M + 31) / 32, (p.N + 31) / 32));
  return launch_kernel(kern, dim3((unsigned)kgroup_tiles(p)), dim3(64 * waves), lds, stream, args);  // a few hundred tiles at most
}

template <class T, class OUT, int KTB, int W, int AMODE, bool TA, bool TB, bool DW>
static hipError_t launch_kgroup_cfg(const GemmParams& p, hipStream_t stream) {
  constexpr int S = 3, LDS = W * S * 64 * KTB;  // (rings of four and five stages: level)
  static_assert(LDS <= 160 * 1024, "LDS budget");
  static std::atomic<bool> configured{LDS <= 64 * 1024};
  return launch_kgroup_grid<std::conditional_t<AMODE == 1, ConvArgs, GemmArgs>, T>(configured, gemm_kgroup_kernel<T, OUT, KTB, S, W, AMODE, TA, TB, DW>, W, LDS, p, stream);
}

// Direct-to-LDS operands (checked by the caller).  Eight waves, a tile to a compute unit, where K keeps them busy; four
// waves, three workgroups to a compute unit, where it does not or where there are more tiles than compute units; and
// 128-byte K tiles for long rows, whose 64-byte pieces two waves would fetch as two halves of a cache line (B^T
// 588 x 128 x 5888 8.4 -> 6.9 us, 83 x 928 x 8048 12.2 -> 10.5).
template <class T, class OUT, int AMODE, bool TA = false, bool TB = false, bool DW = false>
static hipError_t launch_kgroup(const GemmParams& p, hipStream_t stream) {
  const int64_t kbytes = (int64_t)p.K * T::EB;
  if (kgroup_tiles(p) > 256 || kbytes <= 512) return launch_kgroup_cfg<T, OUT, 64, 4, AMODE, TA, TB, DW>(p, stream);
  if constexpr (AMODE == 0)
    if (kbytes >= 4864) return launch_kgroup_cfg<T, OUT, 128, 4, AMODE, TA, TB, DW>(p, stream);
  return launch_kgroup_cfg<T, OUT, 64, 8, AMODE, TA, TB, DW>(p, stream);
}

// Whether the kernel above takes a product (or, `conv`, a convolution) from the others, which would cut K into `splits`.
template <class T, bool TA = false, bool TB = false>
static bool kgroup_takes(const GemmParams& p, bool conv, int splits, bool raw = false) {
  return kgroup_rule({p.M, p.N, p.K, T::EB, conv, !TA, TB, p.ldb * T::EB, splits, p.partial != nullptr, p.Cin, raw});
}

// Whether an uncut product that meets dword_operands takes gemm_dtl_kernel's DW form.
static inline bool dword_tiles(const GemmParams& p, int eb, bool trans_a, bool trans_b) { return dword_tiles_rule(p.M, p.N, (int64_t)p.K * eb, !trans_a && trans_b); }

// Any size, pitch and alignment (at least 16 bytes to a row of a K-strided operand): 16-byte chunks through registers, two
// tiles ahead, into one padded LDS buffer per wave.  AKC, BKC, CONV as for gemm_ragged_kernel.
template <class T, class OUT, int W, bool AKC, bool BKC, bool CONV>
__global__ void __launch_bounds__(64 * W) gemm_kgroup_ragged_kernel(const std::conditional_t<CONV, ConvArgs, GemmArgs> p) {
  using SA = std::conditional_t<CONV, RaggedImage<32, 64>, RaggedMatrix<T, 32, 64, AKC>>;
  using SB = std::conditional_t<CONV, RaggedWeights<32, 64>, RaggedMatrix<T, 32, 64, BKC>>;
  using TA = typename SA::Tile;
  using TB = typename SB::Tile;
  constexpr int PITCH = TA::BYTES + TB::BYTES, KS = RAGGED_KTB / 32;
  static_assert(PITCH >= 4096 && W >= 4, "a wave's sums fit its buffer; four waves run the output stage");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tiles_m = (p.M + 31) / 32, tiles_n = (p.N + 31) / 32;
  int tm, tn;
  tile_coords_mul(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, p.band_magic, tm, tn);
  const int m0 = tm * 32, n0 = tn * 32;
  const int kbytes = walk_bytes<CONV, T::EB>(p);
  const int nkt_total = (kbytes + RAGGED_KTB - 1) / RAGGED_KTB, nkt_whole = CONV ? nkt_total : kbytes / RAGGED_KTB;

  const int om = m0 + (t >> 3), on = n0 + 4 * (t & 7);
  const bool out = t < 256 && om < p.M && on < p.N;
  v4i bias = {0, 0, 0, 0};
  if (out) bias = OUT::prefetch(p, om, on);

  SA a;
  SB b;
  if constexpr (CONV) {
    a.init(p, m0, wave, lane, W);
    b.init(p, n0, wave, lane, W);
  } else {
    a.init(p.A, p.lda, m0, p.M, p.K, wave, lane);
    b.init(p.B, p.ldb, n0, p.N, p.K, wave, lane);
  }
  unsigned char *As = smem + wave * PITCH, *Bs = As + TA::BYTES;
  typename T::accv acc = T::zero();
  auto multiply = [&](const v4i (&xa)[SA::IT], const v4i (&xb)[SB::IT]) {  // one tile: registers -> LDS -> MFMA, within the wave
    TA::store(As, lane, xa);
    TB::store(Bs, lane, xb);
    v4i fa[KS], fb[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      const int kb = ks * 32 + (lane >> 5) * 16;
      fa[ks] = TA::fragment(As, 0, kb, lane);
      fb[ks] = TB::fragment(Bs, 0, kb, lane);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ks++) acc = T::mfma(fb[ks], fa[ks], acc);
  };
  auto fix = [&](v4i (&xa)[SA::IT], v4i (&xb)[SB::IT], const int (&fa)[SA::IT], const int (&fb)[SB::IT]) {
#pragma unroll
    for (int i = 0; i < SA::IT; i++) xa[i] = chunk_apply<CONV>(xa[i], fa[i]);
#pragma unroll
    for (int i = 0; i < SB::IT; i++) xb[i] = chunk_apply<false>(xb[i], fb[i]);
  };
  const int n = nkt_whole > wave ? (nkt_whole - wave + W - 1) / W : 0;  // tiles of this wave, the partial one apart
  v4i ra[2][SA::IT], rb[2][SB::IT];
  int fa[2][SA::IT], fb[2][SB::IT];  // CONV
  if constexpr (!CONV) {
    // the partial last tile, ahead of the others by the wave whose turn it is
    if (nkt_whole < nkt_total && nkt_whole % W == wave) {  // wave-uniform
      typename SA::Last la;
      typename SB::Last lb;
      a.load_last(ra[0], la, nkt_whole - wave);
      b.load_last(rb[0], lb, nkt_whole - wave);
      a.last_fix(ra[0], la);
      b.last_fix(rb[0], lb);
      multiply(ra[0], rb[0]);
    }
  }
  auto fetch = [&](auto sc) {
    constexpr int s = decltype(sc)::value;
    if constexpr (CONV) {
      a.load(ra[s], fa[s]);
      b.load(rb[s], fb[s]);
    } else {
      a.load_whole(ra[s], W * a.step);
      b.load_whole(rb[s], W * b.step);
    }
  };
  auto use = [&](auto sc) {
    constexpr int s = decltype(sc)::value;
    if constexpr (CONV) {
      fix(ra[s], rb[s], fa[s], fb[s]);
    } else {  // of a whole tile, only the last chunk of a K-strided row needs its shift
      if constexpr (!AKC) {
#pragma unroll
        for (int i = 0; i < SA::IT; i++) ra[s][i] = chunk_apply<false>(ra[s][i], a.edge);
      }
      if constexpr (!BKC) {
#pragma unroll
        for (int i = 0; i < SB::IT; i++) rb[s][i] = chunk_apply<false>(rb[s][i], b.edge);
      }
    }
    multiply(ra[s], rb[s]);
  };
  constexpr std::integral_constant<int, 0> s0;
  constexpr std::integral_constant<int, 1> s1;
  if (n >= 2) {  // no request of the steady trips is conditional, so that every wait counts the younger ones
    fetch(s0);
    fetch(s1);
    int k = 0;
#pragma unroll 1
    for (; k + 4 <= n; k += 2) {
      use(s0);
      fetch(s0);
      use(s1);
      fetch(s1);
    }
    use(s0);
    if (k + 2 < n) fetch(s0);
    use(s1);
    if (k + 2 < n) use(s0);
  } else if (n == 1) {
    fetch(s0);
    use(s0);
  }
  kgroup_finish<OUT, W, PITCH>(p, smem, wave, t, acc, om, on, out, bias);
}

template <class T, class OUT, int W, bool AKC, bool BKC, bool CONV>
static hipError_t launch_kgroup_ragged_cfg(const GemmParams& p, hipStream_t stream) {
  constexpr int LDS = W * (RaggedTile<T, 32, 64, AKC>::BYTES + RaggedTile<T, 32, 64, BKC>::BYTES);
  static_assert(LDS <= 160 * 1024, "LDS budget");
  static std::atomic<bool> configured{LDS <= 64 * 1024};
  return launch_kgroup_grid<std::conditional_t<CONV, ConvArgs, GemmArgs>, T>(configured, gemm_kgroup_ragged_kernel<T, OUT, W, AKC, BKC, CONV>, W, LDS, p, stream);
}
template <class T, class OUT, bool AKC, bool BKC, bool CONV = false>
static hipError_t launch_kgroup_ragged(const GemmParams& p, hipStream_t stream) {
  return kgroup_tiles(p) <= 256 ? launch_kgroup_ragged_cfg<T, OUT, 8, AKC, BKC, CONV>(p, stream) : launch_kgroup_ragged_cfg<T, OUT, 4, AKC, BKC, CONV>(p, stream);
}

// The same question for operands of any alignment.
template <class T, bool AKC, bool BKC, bool CONV = false>
static bool kgroup_ragged_takes(const GemmParams& p, int splits) {
  if (CONV && (p.Cin < 1 || p.a_bytes < 16 || p.N < 1)) return false;
  if (!CONV && !((AKC || (int64_t)p.M * T::EB >= 16) && (BKC || (int64_t)p.N * T::EB >= 16))) return false;  // rows of K-strided operands hold a chunk
  return kgroup_ragged_rule({p.M, p.N, p.K, T::EB, CONV, AKC, BKC, p.ldb * T::EB, splits, p.partial != nullptr, p.Cin});
}

}  // namespace ac
