// Operand types and output stages shared by the tiled MFMA kernels for gfx950 (CDNA4): int8 GEMM, int8 implicit-GEMM
// convolution and bf16 GEMM.
#pragma once
#include "common.hpp"
#include <type_traits>

namespace ac {

#define AC_LDS(T, p) ((__attribute__((address_space(3))) T*)(p))

struct TypeI8 {
  static constexpr int EB = 1;  // element bytes
  using accv = v16i;
  static __device__ __forceinline__ accv zero() {
    accv z;
#pragma unroll
    for (int r = 0; r < 16; r++) z[r] = 0;
    return z;
  }
  static __device__ __forceinline__ accv mfma(v4i rowop, v4i colop, accv c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(rowop, colop, c, 0, 0, 0);
  }
  using acc4 = v4i;  // of a 16 x 16 tile
  static __device__ __forceinline__ acc4 mfma(v4i rowop, v4i colop, acc4 c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(rowop, colop, c, 0, 0, 0); }
  // 16 consecutive k (bytes) of one B column, gathered from K-major LDS rows.
  // Within a 16-lane group lane i supplies the address of 8 bytes of row i/2 and
  // receives 8 k-values of column i.
  static __device__ __forceinline__ v4i read_col(const unsigned char* tile, int stride, int k0, int ncol_bytes, int lane) {
    int i = lane & 15;
    const unsigned char* p = tile + (k0 + (i >> 1)) * stride + ncol_bytes + 8 * (i & 1);
    v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, p));
    v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, p + 8 * stride));
    return (v4i){lo[0], lo[1], hi[0], hi[1]};
  }
};

struct TypeBF16 {
  static constexpr int EB = 2;
  using accv = v16f;
  static __device__ __forceinline__ accv zero() {
    accv z;
#pragma unroll
    for (int r = 0; r < 16; r++) z[r] = 0.f;
    return z;
  }
  static __device__ __forceinline__ accv mfma(v4i rowop, v4i colop, accv c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, rowop), __builtin_bit_cast(v8bf, colop), c, 0, 0, 0);
  }
  using acc4 = v4f;
  static __device__ __forceinline__ acc4 mfma(v4i rowop, v4i colop, acc4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, rowop), __builtin_bit_cast(v8bf, colop), c, 0, 0, 0);
  }
  // 8 consecutive k of one B column: lane i of a 16-lane group addresses 4
  // elements of row i/4 and receives 4 k-values of column i.
  static __device__ __forceinline__ v4i read_col(const unsigned char* tile, int stride, int k0, int ncol_bytes, int lane) {
    int i = lane & 15;
    const unsigned char* p = tile + (k0 + (i >> 2)) * stride + ncol_bytes + 8 * (i & 3);
    v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(AC_LDS(v4s, p));
    v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(AC_LDS(v4s, p + 4 * stride));
    v2i l2 = __builtin_bit_cast(v2i, lo), h2 = __builtin_bit_cast(v2i, hi);
    return (v4i){l2[0], l2[1], h2[0], h2[1]};
  }
};

// Epilogue policies -----------------------------------------------------------
// tile(): one 32x32 accumulator tile, whose operand order the policy chooses with SWAP:
//   SWAP (B^T tile as the row operand): register r of lane l is row l % 32, column 8 (r/4) + 4 (l/32) + r % 4:
//     a lane owns runs of 4 consecutive columns of one row.  Right for 1-byte outputs, which pack 4 (and, after
//     a lane exchange, 16) of them per store.
//   !SWAP: register r of lane l is row 8 (r/4) + 4 (l/32) + r % 4, column l % 32: the 32 lanes of a half-wave
//     own 32 consecutive columns of one row, so a 4-byte-per-lane store writes a whole 128-byte row segment.
//     Right for 4-byte outputs: with the swapped order a store instruction scatters 32-byte pieces over 32
//     rows, which the memory system drains at half the rate (measured on a store-bound GEMM).
// tile() receives the tile origin (mrow0, ncol0).

// Applies f(r, m, n) to the 16 accumulators of an unswapped tile: r = register, (m, n) = its coordinates.
template <class F>
static __device__ __forceinline__ void for_each_unswapped(int mrow0, int ncol0, int lane, F f) {
#pragma unroll
  for (int r = 0; r < 16; r++) f(r, mrow0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), ncol0 + (lane & 31));
}

// Stores f(r) for the 16 registers of an unswapped tile, `ld` elements between rows: sixteen plain stores where all 32
// rows exist (wave-uniform; with a guard and an address of its own each they are some 25 instructions apiece).
template <class V, class F>
static __device__ __forceinline__ void store_unswapped(V* base, int64_t ld, int rows, int cols, int mrow0, int ncol0, int lane, F f) {
  const int n = ncol0 + (lane & 31), mb = mrow0 + 4 * (lane >> 5);
  if (n >= cols) return;
  V* dst = base + (int64_t)mb * ld + n;
  if (mrow0 + 32 <= rows) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
#pragma unroll
      for (int e = 0; e < 4; e++) dst[e * ld] = f(4 * q + e);
      dst += 8 * ld;
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; r++) {
      const int dm = 8 * (r >> 2) + (r & 3);
      if (mb + dm < rows) dst[dm * ld] = f(r);
    }
  }
}

// An epilogue that can take a whole wave tile at once declares WAVE_TILE.
template <class E, class = void>
struct has_wave_tile : std::false_type {};
template <class E>
struct has_wave_tile<E, std::void_t<decltype(E::WAVE_TILE)>> : std::true_type {};

struct __attribute__((packed)) Unaligned16 {
  v4i v;
};
// 16 consecutive int8 outputs of a row at any address, the first `valid` of them.
static __device__ __forceinline__ void store_run16(int8_t* dst, v4i o, int valid) {
  if (valid >= 16) {
    ((Unaligned16*)dst)->v = o;
  } else if (valid > 0) {
    uint64_t lo = (uint64_t)(unsigned)o[0] | ((uint64_t)(unsigned)o[1] << 32);
    const uint64_t hi = (uint64_t)(unsigned)o[2] | ((uint64_t)(unsigned)o[3] << 32);
    struct __attribute__((packed)) U8 { uint64_t v; };
    struct __attribute__((packed)) U4 { uint32_t v; };
    struct __attribute__((packed)) U2 { uint16_t v; };
    if (valid & 8) ((U8*)dst)->v = lo, dst += 8, lo = hi;
    if (valid & 4) ((U4*)dst)->v = (uint32_t)lo, dst += 4, lo >>= 32;
    if (valid & 2) ((U2*)dst)->v = (uint16_t)lo, dst += 2, lo >>= 16;
    if (valid & 1) *dst = (int8_t)lo;
  }
}

// int8 output stage: bias, v / 2^shift to nearest (halves to even), saturate, ReLU.
struct EpilogueI8 {
  static constexpr bool SWAP = true;
  static constexpr bool LDS_STAGED = false;
  static __device__ __forceinline__ int requant(int v, int shift, int act) {
    int fl = v >> shift;
    unsigned int rem = (unsigned int)v & ((1u << shift) - 1u);
    unsigned int half = shift > 0 ? (1u << (shift - 1)) : 0u;
    int inc = (shift > 0) && (rem > half || (rem == half && (fl & 1)));
    int q = fl + inc;
    q = q > 127 ? 127 : q;
    q = q < -128 ? -128 : q;
    if (act) q = q < 0 ? 0 : q;
    return q;
  }
  // Columns n .. n + 3 of row m, for a C whose rows are dword-aligned.
  template <class P>
  static __device__ __forceinline__ void store4(const P& p, int m, int n, const int* a) {
    if (m >= p.M || n >= p.N) return;
    int8_t* C = (int8_t*)p.C;
    int v[4];
    const bool full = n + 3 < p.N;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      int b = 0;
      if (p.bias && (full || n + e < p.N)) b = p.bias_ld == 0 ? p.bias[n + e] : p.bias[(int64_t)m * p.bias_ld + n + e];
      v[e] = requant(a[e] + b, p.shift, p.act);
    }
    int8_t* dst = C + (int64_t)m * p.ldc + n;
    if (full) {
      unsigned int w = (unsigned int)(v[0] & 0xff) | ((unsigned int)(v[1] & 0xff) << 8) | ((unsigned int)(v[2] & 0xff) << 16) | ((unsigned int)(v[3] & 0xff) << 24);
      *(unsigned int*)dst = w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (n + e < p.N) dst[e] = (int8_t)v[e];
    }
  }

  // ---- tile-level interface of the direct-to-LDS kernels ----------------------------------------------
  // One 32x32 MFMA tile: lane l holds row m = row0 + l % 32 and, for q = 0..3, columns
  // ncol0 + 8q + 4 (l / 32) + 0..3.
  struct Pre {
    v4i bias[4];  // bias of this lane's 16 columns (row-vector bias only), fetched before the K loop
  };
  // The bias row is read through a bounds-checked buffer of N int32 (no row bias: zero records), so the four
  // loads carry no branches: columns beyond N, and every column when there is no row bias, come back as zeros.
  template <class P>
  static __device__ __forceinline__ void prefetch(const P& p, int ncol0, int lane, Pre& pre) {
    const bool row_bias = p.bias != nullptr && p.bias_ld == 0;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)p.bias, 0, row_bias && p.N < (1 << 29) ? p.N * 4 : 0, 0x00020000);
    const int off = (ncol0 + 4 * (lane >> 5)) * 4;
    if (p.N < (1 << 29)) {  // wave-uniform; byte offsets fit the signed 32-bit buffer arithmetic
#pragma unroll
      for (int q = 0; q < 4; q++) pre.bias[q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + 32 * q, 0, 0);
    } else {
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int n = ncol0 + 8 * q + 4 * (lane >> 5);
        pre.bias[q] = (v4i){0, 0, 0, 0};
        if (row_bias && n + 3 < p.N) pre.bias[q] = (v4i){p.bias[n], p.bias[n + 1], p.bias[n + 2], p.bias[n + 3]};
      }
    }
  }
  // Fast form of requant() for 1 <= shift <= 23: floor((t + 2^(shift-1) - 1 + bit) / 2^shift) with bit = bit
  // `shift` of t rounds halves to even.  The rounding shift is monotone, so the output clamp is taken on the way
  // in: t is clamped to [lo, hi] with hi = 127 * 2^shift + 2^(shift-1) - 1, the largest t that still rounds to
  // 127, and lo = -128 * 2^shift, which rounds to -128 exactly (0 with ReLU: every negative t ends as 0), which
  // also keeps the rounding add inside int32 and makes both activations the same code.
  struct FastQuant {
    int shift, rnd, lo, hi;
    float scale, lo_f, hi_f;  // 2^-shift and the bounds as fp32 (exact for shifts up to 17)
  };
  static __device__ __forceinline__ FastQuant fast_quant(int shift, int act) {
    const int rnd = (1 << (shift - 1)) - 1, lo = act ? 0 : -128 * (1 << shift), hi = (127 << shift) + rnd;
    return {shift, rnd, lo, hi, __builtin_ldexpf(1.f, -shift), (float)lo, (float)hi};
  }
  // FLOAT_ROUND (shift <= 17): the bounds are at most 2^24 in magnitude, so they and everything between them are
  // exact in fp32, and the conversion of a sum outside them (rounded, but monotone) stays outside them: the sum is
  // converted first and clamped as a float (one median instruction), and one fused multiply-add
  // c * 2^-shift + 1.5 * 2^23 rounds the quotient to an integer, halves to even (the result lies in [2^23, 2^24),
  // where fp32 steps by 1 and the constant is even): the low byte of its bit pattern is the two's-complement
  // output.  Three VALU instructions per value; only the low byte of the returned word is meaningful.
  // Otherwise (shifts 18..23): clamp (a maximum and a minimum: with bounds that are not constants the compiler
  // cannot form the integer median), bit extract, three-operand add, shift.
  template <bool FLOAT_ROUND = false>
  static __device__ __forceinline__ int requant_fast(int t, const FastQuant& f) {
    if constexpr (FLOAT_ROUND) {
      const float c = __builtin_amdgcn_fmed3f((float)t, f.lo_f, f.hi_f);
      return __builtin_bit_cast(int, __builtin_fmaf(c, f.scale, 12582912.f));
    } else {
      int c = t < f.lo ? f.lo : t;
      c = c > f.hi ? f.hi : c;
      const int bit = (int)__builtin_amdgcn_ubfe((unsigned)c, (unsigned)f.shift, 1u);
      return (c + bit + f.rnd) >> f.shift;
    }
  }
  // The low bytes of four words in one dword (v0 lowest).
  static __device__ __forceinline__ unsigned pack4(int v0, int v1, int v2, int v3) {
    const unsigned lo = __builtin_amdgcn_perm((unsigned)v1, (unsigned)v0, 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm((unsigned)v3, (unsigned)v2, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
  }
  // The 16 values of one lane (accumulator + bias), quantised and packed four to a dword -> 16 output bytes in
  // column order after the lane exchange: lanes l and l + 32 hold interleaved 4-byte pieces of the same row.
  // Swapping the upper half of d[0] (d[1]) with the lower half of d[2] (d[3]) leaves 16 consecutive bytes in every
  // lane: columns 0..15 in lanes 0..31, columns 16..31 in lanes 32..63, so a row leaves as two whole 16-byte stores.
  static __device__ __forceinline__ v4i exchange16(const unsigned* d) {
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    const v2u s02 = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false);
    const v2u s13 = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
    return (v4i){(int)s02[0], (int)s02[1], (int)s13[0], (int)s13[1]};
  }
  // Any shift / activation (requant).
  static __device__ __forceinline__ v4i quant16(const int* t, int shift, int act) {
    unsigned d[4];
#pragma unroll
    for (int q = 0; q < 4; q++) d[q] = pack4(requant(t[4 * q], shift, act), requant(t[4 * q + 1], shift, act), requant(t[4 * q + 2], shift, act), requant(t[4 * q + 3], shift, act));
    return exchange16(d);
  }
  // Fast form.
  template <bool FLOAT_ROUND = false>
  static __device__ __forceinline__ v4i quant16(const int* t, const FastQuant& f) {
    unsigned d[4];
#pragma unroll
    for (int q = 0; q < 4; q++)
      d[q] = pack4(requant_fast<FLOAT_ROUND>(t[4 * q], f), requant_fast<FLOAT_ROUND>(t[4 * q + 1], f), requant_fast<FLOAT_ROUND>(t[4 * q + 2], f), requant_fast<FLOAT_ROUND>(t[4 * q + 3], f));
    return exchange16(d);
  }
  // Fast form, the rounding picked by the shift (wave-uniform).
  static __device__ __forceinline__ v4i quant16_by_shift(const int* t, const FastQuant& f) {
    return f.shift <= 17 ? quant16<true>(t, f) : quant16<false>(t, f);
  }
  // The whole wave tile, TM x TN blocks of 32 x 32, when every block takes 16-byte stores, the bias is a row or
  // absent and the shift has the fast form: one decision per wave tile and straight-line code for its blocks (as
  // separate calls of tile() every block carries the whole decision tree, and the output stage of a 256 x 256
  // tile ran through some 90 KB of code).  BIASED as in tile().
  static constexpr bool WAVE_TILE = true;
  // acc_of(i, j) and pre_of(j) give block (i, j)'s accumulators and column block j's prefetched bias.
  template <bool BIASED, int TM, int TN, class ACC_OF, class PRE_OF, class P>
  static __device__ __forceinline__ void wave_blocks(const P& p, int mrow0, int ncol0, ACC_OF acc_of, int lane, int esplit, PRE_OF pre_of) {
    int8_t* C = (int8_t*)p.C;
    const bool fast = ncol0 + 32 * TN <= p.N && (p.bias == nullptr || p.bias_ld == 0) && p.shift >= 1 && p.shift <= 23;
    if (fast) {  // wave-uniform
      const FastQuant f = fast_quant(p.shift, p.act);
      auto blocks = [&](auto float_round) {
#pragma unroll
        for (int i = 0; i < TM; i++) {
          const int m = mrow0 + 32 * i + (lane & 31);
          int8_t* dst = C + (int64_t)m * p.ldc + ncol0 + 16 * (lane >> 5);
#pragma unroll
          for (int j = 0; j < TN; j++) {
            int t[16];
#pragma unroll
            for (int r = 0; r < 16; r++) t[r] = BIASED ? acc_of(i, j)[r] : acc_of(i, j)[r] + pre_of(j).bias[r >> 2][r & 3];  // no bias: the prefetch returned zeros
            const v4i o = quant16<decltype(float_round)::value>(t, f);
            if (m < p.M) ((Unaligned16*)(dst + 32 * j))->v = o;
          }
        }
      };
      if (p.shift <= 17) blocks(std::true_type{});
      else blocks(std::false_type{});
    } else {
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) tile<BIASED>(p, mrow0 + 32 * i, ncol0 + 32 * j, acc_of(i, j), lane, esplit, pre_of(j));
    }
  }
  template <bool BIASED = false, int TM, int TN, class ACC, class P>
  static __device__ __forceinline__ void wave_tile(const P& p, int mrow0, int ncol0, const ACC (&acc)[TM][TN], int lane, int esplit, const Pre (&pre)[TN]) {
    wave_blocks<BIASED, TM, TN>(p, mrow0, ncol0, [&](int i, int j) -> const ACC& { return acc[i][j]; }, lane, esplit, [&](int j) -> const Pre& { return pre[j]; });
  }
  // The wave tile as TM x TN tiles of 16 x 16, for shifts 1..17 and no bias or a row of it: lane l holds of each tile the row
  // l % 16 and the columns 4 (l / 16) .. + 3.  Four tiles of a row are quantised to a dword a lane each and exchanged between
  // registers and lane groups (a 4 x 4 transpose), after which lane group g stores tile g, 16 bytes of a row a lane.
  struct Pre16 {
    v4i bias;  // of the lane's four columns
  };
  static bool takes16(int shift, const void* bias, int64_t bias_ld) { return shift >= 1 && shift <= 17 && (bias == nullptr || bias_ld == 0); }
  template <int TM, int TN, class P>
  static __device__ __forceinline__ void wave_tile(const P& p, int mrow0, int ncol0, const v4i (&acc)[TM][TN], int lane, int, const Pre16 (&pre)[TN]) {
    static_assert(TN % 4 == 0, "four tiles at a time");
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    const FastQuant f = fast_quant(p.shift, p.act);
    int8_t* dst = (int8_t*)p.C + (int64_t)(mrow0 + (lane & 15)) * p.ldc + ncol0 + 16 * (lane >> 4);
    const int64_t down = 16 * p.ldc;
    const int rows = p.M - mrow0 - (lane & 15), cols = p.N - ncol0 - 16 * (lane >> 4);
    auto groups = [&](auto whole) {
#pragma unroll
      for (int i = 0; i < TM; i++) {
#pragma unroll
        for (int j = 0; j < TN; j += 4) {
          unsigned d[4];
#pragma unroll
          for (int s = 0; s < 4; s++) {
            const v4i t = acc[i][j + s] + pre[j + s].bias;  // no bias: zeros
            d[s] = pack4(requant_fast<true>(t[0], f), requant_fast<true>(t[1], f), requant_fast<true>(t[2], f), requant_fast<true>(t[3], f));
          }
          const v2u a = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false), b = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
          const v2u lo = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false), hi = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
          const v4i o = {(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
          if constexpr (decltype(whole)::value) ((Unaligned16*)(dst + 16 * j))->v = o;
          else if (16 * i < rows) store_run16(dst + 16 * j, o, cols - 16 * j);
          __builtin_amdgcn_sched_barrier(0);  // or a tile's worth of them is in flight at once, out of registers
        }
        dst += down;
      }
    };
    if (mrow0 + 16 * TM <= p.M && ncol0 + 16 * TN <= p.N) groups(std::true_type{});  // wave-uniform
    else groups(std::false_type{});
  }
  // A column of TM blocks with one bias block.
  template <bool BIASED = false, int TM, class ACC, class P>
  static __device__ __forceinline__ void wave_column(const P& p, int mrow0, int ncol0, const ACC (&acc)[TM], int lane, const Pre& pre) {
    wave_blocks<BIASED, TM, 1>(p, mrow0, ncol0, [&](int i, int) -> const ACC& { return acc[i]; }, lane, 0, [&](int) -> const Pre& { return pre; });
  }
  // BIASED: the accumulators already hold the bias (a kernel that starts its sums from the bias row).
  template <bool BIASED = false, class ACC, class P>
  static __device__ __forceinline__ void tile(const P& p, int mrow0, int ncol0, const ACC& acc, int lane, int, const Pre& pre) {
    const int m = mrow0 + (lane & 31);
    if (m >= p.M || ncol0 >= p.N) return;
    int8_t* C = (int8_t*)p.C;
    const bool row_bias = p.bias && p.bias_ld == 0;
    int t[16];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int n = ncol0 + 8 * q + 4 * (lane >> 5);
#pragma unroll
      for (int e = 0; e < 4; e++) {
        int b = 0;
        if constexpr (!BIASED) {
          b = row_bias ? pre.bias[q][e] : 0;
          if (p.bias && !row_bias) b = p.bias[(int64_t)m * p.bias_ld + (n + e < p.N ? n + e : p.N - 1)];
        }
        t[4 * q + e] = acc[4 * q + e] + b;
      }
    }
    const v4i o = p.shift >= 1 && p.shift <= 23 ? quant16_by_shift(t, fast_quant(p.shift, p.act)) : quant16(t, p.shift, p.act);
    const int n = ncol0 + 16 * (lane >> 5);
    store_run16(C + (int64_t)m * p.ldc + n, o, p.N - n);
  }
};

// The same output stage for a C of any alignment and pitch: after the exchange a lane holds 16 consecutive columns of
// its row and stores them with one unaligned store (one byte per lane and store, on unswapped tiles, is sixteen stores
// with their guards and addresses).
struct EpilogueI8Any {
  static constexpr bool SWAP = true;
  struct Pre {};
  template <class P>
  static __device__ __forceinline__ void one(const P& p, int m, int n, int v) {
    if (p.bias) v += p.bias_ld == 0 ? p.bias[n] : p.bias[(int64_t)m * p.bias_ld + n];
    ((int8_t*)p.C)[(int64_t)m * p.ldc + n] = (int8_t)EpilogueI8::requant(v, p.shift, p.act);
  }
  template <class ACC, class P>
  static __device__ __forceinline__ void tile(const P& p, int mrow0, int ncol0, const ACC& acc, int lane, int, const Pre&) {
    if (ncol0 >= p.N) return;
    const int m = mrow0 + (lane & 31), half = lane >> 5;
    int v[16];
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = acc[r];
    if (p.bias) {
      // a row is read through a bounds-checked buffer of N values, one of the rows of a matrix (or a row of more than
      // 2^29 values) with a guard on every value: columns beyond N are not stored, whatever is added to them
      if (p.bias_ld == 0 && p.N < (1 << 29)) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)p.bias, 0, p.N * 4, 0x00020000);
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] += __builtin_amdgcn_raw_buffer_load_b32(rsrc, (ncol0 + 8 * (r >> 2) + 4 * half + (r & 3)) * 4, 0, 0);
      } else {
        const int32_t* const row = p.bias + (p.bias_ld != 0 ? (int64_t)(m < p.M ? m : p.M - 1) * p.bias_ld : 0);
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int n = ncol0 + 8 * (r >> 2) + 4 * half + (r & 3);
          v[r] += row[n < p.N ? n : p.N - 1];
        }
      }
    }
    const v4i o = p.shift >= 1 && p.shift <= 23 ? EpilogueI8::quant16_by_shift(v, EpilogueI8::fast_quant(p.shift, p.act)) : EpilogueI8::quant16(v, p.shift, p.act);
    const int n = ncol0 + 16 * half;
    if (m < p.M) store_run16((int8_t*)p.C + (int64_t)m * p.ldc + n, o, p.N - n);
  }
};

// Split-K partial sums: raw int32 accumulators of K slice `split` go to partial[split][M][N]; the output stage
// runs in splitk_reduce_i8_kernel once every slice has been written.
struct EpiloguePartialI32 {
  static constexpr bool SWAP = false;
  static constexpr bool LDS_STAGED = true;  // the workspace is 16-byte aligned and N a multiple of 16 on this path
  static constexpr bool STAGED_READS = false;
  typedef int StagedValue;
  template <class P>
  static __device__ __forceinline__ int staged_in(const P&, int a) { return a; }
  template <class P>
  static __device__ __forceinline__ void staged_out(const P& p, int m, int n, v4i o, int split, int) {
    *(v4i*)(p.partial + ((int64_t)split * p.M + m) * p.N + n) = o;
  }
  template <class P>
  static __device__ __forceinline__ int staged_add(const P&, int) { return 0; }
  struct Pre {};
  template <class P>
  static __device__ __forceinline__ void prefetch(const P&, int, int, Pre&) {}
  template <class ACC, class P>
  static __device__ __forceinline__ void tile(const P& p, int mrow0, int ncol0, const ACC& acc, int lane, int split, const Pre&) {
    store_unswapped(p.partial + (int64_t)split * p.M * p.N, p.N, p.M, p.N, mrow0, ncol0, lane, [&](int r) { return acc[r]; });
  }
};

// Raw accumulator output (the accumulator-type read of the paper's accelerator: no scaling, no activation):
// C32[m][n] = acc + bias, int32, row stride ldc.
struct EpilogueRawI32 {
  static constexpr bool SWAP = false;
  static constexpr bool LDS_STAGED = true;  // C is 16-byte aligned with ldc a multiple of 4 on this path
  static constexpr bool STAGED_READS = true;
  typedef int StagedValue;
  template <class P>
  static __device__ __forceinline__ int staged_in(const P&, int a) { return a; }
  template <class P>
  static __device__ __forceinline__ void staged_out(const P& p, int m, int n, v4i o, int, v4i add) {
    *(v4i*)((int32_t*)p.C + (int64_t)m * p.ldc + n) = o + add;
  }
  // A bias matrix is read element by element, a row once (staged_add).
  template <class P>
  static __host__ __device__ __forceinline__ bool staged_reads(const P& p) { return p.bias != nullptr && p.bias_ld != 0; }
  template <class P>
  static __device__ __forceinline__ v4i staged_read(const P& p, int m, int n) {
    const int32_t* b = p.bias + (int64_t)m * p.bias_ld + n;  // only 4-byte aligned
    return (v4i){b[0], b[1], b[2], b[3]};
  }
  // The bias row's values of columns n .. n + 3 (N is a multiple of 4 on this path), or zeros.  They are waited for here: the
  // compiler would wait at a store, where it knows neither whether they were loaded nor how many requests are younger.
  template <class P>
  static __device__ __forceinline__ v4i staged_add(const P& p, int n) {
    v4i row = {0, 0, 0, 0};
    if (p.bias != nullptr && p.bias_ld == 0 && n < p.N) {
      const int32_t* b = p.bias + n;
      row = (v4i){b[0], b[1], b[2], b[3]};
      asm volatile("" : "+v"(row));
    }
    return row;
  }
  struct Pre {};
  template <class P>
  static __device__ __forceinline__ void prefetch(const P&, int, int, Pre&) {}
  template <class P>
  static __device__ __forceinline__ void one(const P& p, int m, int n, int v) {
    if (p.bias) v += p.bias_ld == 0 ? p.bias[n] : p.bias[(int64_t)m * p.bias_ld + n];
    ((int32_t*)p.C)[(int64_t)m * p.ldc + n] = v;
  }
  template <class ACC, class P>
  static __device__ __forceinline__ void tile(const P& p, int mrow0, int ncol0, const ACC& acc, int lane, int, const Pre&) {
    if (p.bias != nullptr && p.bias_ld != 0) {
      for_each_unswapped(mrow0, ncol0, lane, [&](int r, int m, int n) {
        if (m < p.M && n < p.N) one(p, m, n, acc[r]);
      });
      return;
    }
    const int n = ncol0 + (lane & 31);
    const int bias = p.bias && n < p.N ? p.bias[n] : 0;
    store_unswapped((int32_t*)p.C, p.ldc, p.M, p.N, mrow0, ncol0, lane, [&](int r) { return acc[r] + bias; });
  }
};

// fp32 output: C = alpha * acc + beta * C (C read only when beta != 0).
struct EpilogueF32 {
  static constexpr bool SWAP = false;
  // The direct-to-LDS kernels hand over 4-byte outputs through an LDS transpose: staged_in() is applied to every
  // accumulator on its way into LDS, staged_out() receives four consecutive columns of one row and what is added to them:
  // staged_read()'s values of the same elements where staged_reads() says that there are any, otherwise staged_add()'s, which
  // are the same in every row.
  static constexpr bool LDS_STAGED = true;
  static constexpr bool STAGED_READS = true;
  typedef float StagedValue;
  template <class P>
  static __device__ __forceinline__ float staged_in(const P& p, float a) { return p.alpha * a; }
  template <class P>
  static __device__ __forceinline__ void staged_out(const P& p, int m, int n, v4f o, int, int) {
    *(v4f*)((float*)p.C + (int64_t)m * p.ldc + n) = o;
  }
  template <class P>
  static __device__ __forceinline__ void staged_out(const P& p, int m, int n, v4f o, int, v4f old) {
    *(v4f*)((float*)p.C + (int64_t)m * p.ldc + n) = o + p.beta * old;
  }
  template <class P>
  static __host__ __device__ __forceinline__ bool staged_reads(const P& p) { return p.beta != 0.f; }
  template <class P>
  static __device__ __forceinline__ v4f staged_read(const P& p, int m, int n) { return *(const v4f*)((const float*)p.C + (int64_t)m * p.ldc + n); }
  template <class P>
  static __device__ __forceinline__ int staged_add(const P&, int) { return 0; }
  struct Pre {};
  template <class P>
  static __device__ __forceinline__ void prefetch(const P&, int, int, Pre&) {}
  template <class P>
  static __device__ __forceinline__ void one(const P& p, int m, int n, float v) {
    float* dst = (float*)p.C + (int64_t)m * p.ldc + n;
    float o = p.alpha * v;
    if (p.beta != 0.f) o += p.beta * *dst;
    *dst = o;
  }
  template <class ACC, class P>
  static __device__ __forceinline__ void tile(const P& p, int mrow0, int ncol0, const ACC& acc, int lane, int, const Pre&) {
    if (p.beta == 0.f) {
      store_unswapped((float*)p.C, p.ldc, p.M, p.N, mrow0, ncol0, lane, [&](int r) { return p.alpha * acc[r]; });
      return;
    }
    for_each_unswapped(mrow0, ncol0, lane, [&](int r, int m, int n) {
      if (m < p.M && n < p.N) one(p, m, n, acc[r]);
    });
  }
};

// Split-K output of the fp32 epilogue: every K slice adds alpha * (its partial product) into C with the
// hardware fp32 atomic add; C was set to beta * C by scale_c_f32_kernel before the slices run.  The order in
// which slices arrive is not fixed, so the last bits of a sum may differ between runs.
struct EpilogueAtomicF32 {
  static constexpr bool SWAP = false;
  static constexpr bool LDS_STAGED = false;
  struct Pre {};
  template <class P>
  static __device__ __forceinline__ void prefetch(const P&, int, int, Pre&) {}
  template <class ACC, class P>
  static __device__ __forceinline__ void tile(const P& p, int mrow0, int ncol0, const ACC& acc, int lane, int, const Pre&) {
    for_each_unswapped(mrow0, ncol0, lane, [&](int r, int m, int n) {
      if (m < p.M && n < p.N) unsafeAtomicAdd((float*)p.C + (int64_t)m * p.ldc + n, p.alpha * acc[r]);
    });
  }
};

// Split-K partial products in fp32: slice `split` stores its raw accumulators to partial[split][M][N] (the
// int32 workspace pointer reinterpreted); splitk_reduce_f32_kernel sums the slices in slice order and applies
// alpha / beta, so the result does not depend on which slice finishes first.
struct EpiloguePartialF32 {
  static constexpr bool SWAP = false;
  static constexpr bool LDS_STAGED = true;  // the workspace is 16-byte aligned and N a multiple of 8 on this path
  static constexpr bool STAGED_READS = false;
  typedef float StagedValue;
  template <class P>
  static __device__ __forceinline__ float staged_in(const P&, float a) { return a; }
  template <class P>
  static __device__ __forceinline__ void staged_out(const P& p, int m, int n, v4f o, int split, int) {
    *(v4f*)((float*)p.partial + ((int64_t)split * p.M + m) * p.N + n) = o;
  }
  template <class P>
  static __device__ __forceinline__ int staged_add(const P&, int) { return 0; }
  struct Pre {};
  template <class P>
  static __device__ __forceinline__ void prefetch(const P&, int, int, Pre&) {}
  template <class ACC, class P>
  static __device__ __forceinline__ void tile(const P& p, int mrow0, int ncol0, const ACC& acc, int lane, int split, const Pre&) {
    for_each_unswapped(mrow0, ncol0, lane, [&](int r, int m, int n) {
      if (m < p.M && n < p.N) ((float*)p.partial)[((int64_t)split * p.M + m) * p.N + n] = acc[r];
    });
  }
};

}  // namespace ac
