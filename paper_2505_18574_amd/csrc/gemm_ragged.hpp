// Tiled MFMA GEMM / implicit-GEMM convolution for operands of any size, pitch and alignment: whatever the
// direct-to-LDS kernels (gemm_dtl.hpp) do not take, beyond the few tiles that gemm_kgroup.hpp shares.  int8 and bf16, either
// operand transposed in memory, and convolutions with any channel count.
//
// Every 16-byte chunk of an operand tile comes in with ONE vector load, wherever it starts (a vector load takes any
// byte address; a chunk fetched byte by byte is sixteen loads and as many waits on the address unit, which is what
// bounded the kernel this one replaces).  A chunk that would reach past the end of its row or of the buffer is loaded
// from the nearest address at which 16 bytes exist and is shifted and masked in registers on its way into LDS, so no
// load is conditional and the pipeline never depends on where a tile lies:
//   K-contiguous operand (A, B^T): rows beyond the extent are clamped to the last row (their products are never
//     stored); bytes beyond K are zeroed, which only the last K tile has.
//   K-strided operand (B, A^T): k-rows beyond K are zeroed; the chunk across the row's end is shifted, the bytes that
//     follow the last column belong to outputs that are never stored.
//   Convolution input: K is ordered (kh, kw, ci), so the KW * Cin bytes of one kernel row are contiguous in the NHWC
//     image.  The kernel pads that run to whole chunks (the weight rows of the padding are zeroed, so whatever the
//     image bytes there are does not matter) and a chunk then lies in one image row: one load, plus a mask where the
//     window hangs over the left or right edge.
//
// global (16 bytes per lane, R tiles ahead in registers) -> LDS (two buffers, padded rows) -> MFMA, one barrier per K
// tile; the LDS write of a tile runs under the reads and products of the one before.  Two tiles in registers are enough:
// four lose what their longer code costs (bf16 1000 x 1000 x 1022 10.4 us with two, 11.4 with four before the trips
// were overlapped, int8 1000^3 7.7 and 8.6 after).
//
// Bound: the chain of a trip (barrier, LDS reads, products) for the sizes that fill the chip once, 0.26 us a K tile
// against 0.12 on the direct-to-LDS kernels, and some 1.3 us more set-up; LDS writes beyond (some 72 bytes per clock
// and compute unit).  Overlapped trips, the partial tile ahead of the pipeline and 16-byte stores of int8 outputs,
// before and after: int8 1000^3 10.0 -> 7.7, 72 x 252 x 100 5.2 -> 4.2, 364 x 20 x 920 8.8 -> 7.0, 1516 x 1764 x 56
// 9.2 -> 6.1; bf16 1023 x 1537 x 1021 19.2 -> 15.0, 712 x 101 x 204 7.5 -> 6.1, 999 x 999 x 333 9.5 -> 7.8.
#pragma once
#include "gemm_dtl.hpp"

namespace ac {

struct __attribute__((packed, aligned(4))) Dwords16 {
  v4i v;
};
static __device__ __forceinline__ v4i load16_any(const unsigned char* p) { return ((const Unaligned16*)p)->v; }

// What has to happen to a loaded chunk on its way into LDS: shift its bytes down by `s` (up when negative) and keep
// bytes [lo, hi).  One word: s + 16 | lo << 8 | hi << 16.
constexpr int CHUNK_AS_IS = 16 | (16 << 16);
static __device__ __forceinline__ int chunk_fix(int s, int lo, int hi) { return (s + 16) | (lo << 8) | (hi << 16); }
struct Chunk {
  uint64_t a, b;
};
static __device__ __forceinline__ Chunk chunk_down(Chunk c, int bytes) {  // 0 .. 16; zeros come in at the top
  const bool big = bytes >= 8;
  const int n = 8 * (bytes & 7);
  const uint64_t lo = big ? c.b : c.a, hi = big ? 0 : c.b;
  const bool all = bytes >= 16;
  return {all ? 0 : (lo >> n) | ((hi << 1) << (63 - n)), all ? 0 : hi >> n};
}
static __device__ __forceinline__ Chunk chunk_up(Chunk c, int bytes) {
  const bool big = bytes >= 8;
  const int n = 8 * (bytes & 7);
  const uint64_t hi = big ? c.a : c.b, lo = big ? 0 : c.a;
  const bool all = bytes >= 16;
  return {all ? 0 : lo << n, all ? 0 : (hi << n) | ((lo >> 1) >> (63 - n))};
}
// BOTH_ENDS: the fix may shift upwards and cut at the low end (a convolution window over the left edge); otherwise it
// shifts down only and lo == 0.
template <bool BOTH_ENDS>
static __device__ __forceinline__ v4i chunk_apply(v4i v, int fix) {
  if (fix != CHUNK_AS_IS) {
    const int s = (fix & 0xff) - 16, lo = (fix >> 8) & 0xff, hi = fix >> 16;
    Chunk c = {(uint64_t)(unsigned)v[0] | ((uint64_t)(unsigned)v[1] << 32), (uint64_t)(unsigned)v[2] | ((uint64_t)(unsigned)v[3] << 32)};
    c = chunk_down(c, BOTH_ENDS && s < 0 ? 0 : s);
    if constexpr (BOTH_ENDS) c = chunk_up(c, s < 0 ? -s : 0);
    const Chunk m = chunk_down({~(uint64_t)0, ~(uint64_t)0}, 16 - hi);
    c.a &= m.a, c.b &= m.b;
    if constexpr (BOTH_ENDS) {
      const Chunk l = chunk_up({~(uint64_t)0, ~(uint64_t)0}, lo);
      c.a &= l.a, c.b &= l.b;
    }
    v = (v4i){(int)(unsigned)c.a, (int)(unsigned)(c.a >> 32), (int)(unsigned)c.b, (int)(unsigned)(c.b >> 32)};
  }
  return v;
}

constexpr int RAGGED_KTB = 128;  // bytes of K per tile

// One operand tile.  EXT: tile extent along m (or n).  KC: K-contiguous in memory, tile [EXT][KTB]; otherwise
// K-strided, tile [KTB / EB k-rows][EXT * EB bytes].  Rows carry 16 bytes of padding, as in the direct reads of
// TypeI8::read_col / TypeBF16::read_col: both fragment reads are then free of bank conflicts.
template <class T, int EXT, int THREADS, bool KC>
struct RaggedTile {
  static constexpr int EB = T::EB;
  static constexpr int ROW = KC ? RAGGED_KTB : EXT * EB;
  static constexpr int ROWS = KC ? EXT : RAGGED_KTB / EB;
  static constexpr int STRIDE = ROW + 16;
  static constexpr int BYTES = ROWS * STRIDE;
  static constexpr int CPR = ROW / 16;              // chunks per row
  static constexpr int RPP = THREADS / CPR;         // rows per pass of the workgroup
  static constexpr int IT = ROWS / RPP;             // chunks per thread
  static_assert(THREADS % CPR == 0 && ROWS % RPP == 0 && IT >= 1, "tile / thread mismatch");
  static __device__ __forceinline__ void store(unsigned char* tile, int t, const v4i (&reg)[IT]) {
    const int cc = t % CPR, r0 = t / CPR;
#pragma unroll
    for (int i = 0; i < IT; i++) *(v4i*)(tile + (r0 + i * RPP) * STRIDE + cc * 16) = reg[i];
  }
  // MFMA operand: rows (columns) off .. off + 31 of the tile, this lane's K bytes kb .. kb + 15
  static __device__ __forceinline__ v4i fragment(const unsigned char* tile, int off, int kb, int lane) {
    if constexpr (KC) return *(const v4i*)(tile + (off + (lane & 31)) * STRIDE + kb);
    else return T::read_col(tile, STRIDE, kb / EB, (off + 16 * ((lane >> 4) & 1)) * EB, lane);
  }
};

// Source of a matrix operand (see the head of the file).
template <class T, int EXT, int THREADS, bool KC>
struct RaggedMatrix {
  using Tile = RaggedTile<T, EXT, THREADS, KC>;
  static constexpr int EB = T::EB, IT = Tile::IT;
  const unsigned char *base, *last;  // first byte of the matrix, last address with 16 bytes behind it (the launcher makes sure there is one)
  const unsigned char* ptr[IT];      // this thread's chunks of the next tile to load
  int64_t step;                      // bytes from one K tile to the next
  int kb, kbytes;                    // KC: byte of K of this thread's chunk in the first tile; bytes of K
  int k, K;                          // !KC: k-row of its first chunk in the first tile; K
  int edge;                          // !KC: the fix of this thread's column (the same for every k-row)

  __device__ __forceinline__ void init(const void* p, int64_t ld_elems, int origin, int extent, int K_, int kt0, int t) {
    base = (const unsigned char*)p;
    const int64_t ld = ld_elems * EB;
    const int cc = t % Tile::CPR, r0 = t / Tile::CPR;
    K = K_, kbytes = K_ * EB;
    kb = k = 0, edge = CHUNK_AS_IS;
    if constexpr (KC) {
      last = base + (int64_t)(extent - 1) * ld + kbytes - 16;
      step = RAGGED_KTB;
      kb = kt0 * RAGGED_KTB + cc * 16;
#pragma unroll
      for (int i = 0; i < IT; i++) {
        const int row = origin + r0 + i * Tile::RPP;
        ptr[i] = base + (int64_t)(row < extent ? row : extent - 1) * ld + kb;
      }
    } else {
      last = base + (int64_t)(K_ - 1) * ld + (int64_t)extent * EB - 16;
      step = (int64_t)(RAGGED_KTB / EB) * ld;
      k = kt0 * (RAGGED_KTB / EB) + r0;
      int64_t col = (int64_t)origin * EB + cc * 16;
      const int64_t over = col + 16 - (int64_t)extent * EB;
      if (over >= 16) col = 0;  // outside the matrix: any column does
      else if (over > 0 && col >= over) edge = chunk_fix((int)over, 0, 16), col -= over;
      // over > col: a row of fewer than 16 bytes, whose 16 bytes reach into the next row (or, at the end, see guarded())
#pragma unroll
      for (int i = 0; i < IT; i++) ptr[i] = base + (int64_t)(k + i * Tile::RPP) * ld + col;
    }
  }
  // 16 bytes at an address that need not have 16 bytes behind it
  __device__ __forceinline__ v4i guarded(const unsigned char* p, int lo, int hi, int& fix) const {
    const unsigned char* q = p > last ? last : p;
    const int64_t s = p - q;  // 16 and more only for a chunk of which nothing is kept
    fix = s >= 16 ? chunk_fix(0, 0, 0) : chunk_fix((int)s, lo, hi);
    return load16_any(q);
  }
  // the next tile in order, which must lie inside K with every row of it at least 16 bytes long; the one after it lies
  // `advance` bytes further on
  __device__ __forceinline__ void load_whole(v4i (&reg)[IT], int64_t advance) {
#pragma unroll
    for (int i = 0; i < IT; i++) {
      reg[i] = load16_any(ptr[i]);
      ptr[i] += advance;
    }
  }
  // any tile: the one `ahead` tiles after the first
  __device__ __forceinline__ void load_any(v4i (&reg)[IT], int (&fix)[IT], int ahead) const {
    const int64_t off = ahead * step;
#pragma unroll
    for (int i = 0; i < IT; i++) {
      if constexpr (KC) {
        const int valid = kbytes - (kb + ahead * RAGGED_KTB);
        reg[i] = guarded(valid > 0 ? ptr[i] + off : base, 0, valid < 0 ? 0 : (valid < 16 ? valid : 16), fix[i]);
      } else {
        const bool in = k + ahead * (RAGGED_KTB / EB) + i * Tile::RPP < K;
        reg[i] = guarded(in ? ptr[i] + off : base, 0, in ? 16 : 0, fix[i]);
        // the shift of the row's last chunk; it was loaded 16 bytes before the row's end, which is never beyond `last`
        if (in && edge != CHUNK_AS_IS) fix[i] = edge;
      }
    }
  }
  // The partial last tile, `ahead` tiles after the next whole one, where every row is at least 16 bytes long: all chunks are
  // requested, then brought into shape by last_fix().  A K-contiguous operand can leave the buffer in its last row only
  // (the chunk is then loaded where 16 bytes exist and shifted), and its lanes' chunks all end at the same byte of K;
  // a K-strided one has whole rows or rows of zeros.
  struct Last {
    int shift[KC ? IT : 1];  // KC: bytes the chunk was loaded too early
    int ahead;
  };
  __device__ __forceinline__ void load_last(v4i (&reg)[IT], Last& l, int ahead) const {
    const int64_t off = ahead * step;
    l.ahead = ahead;
#pragma unroll
    for (int i = 0; i < IT; i++) {
      if constexpr (KC) {
        const unsigned char *p = ptr[i] + off, *q = p > last ? last : p;
        l.shift[i] = (int)(p - q);
        reg[i] = load16_any(q);
      } else {
        reg[i] = load16_any(k + ahead * (RAGGED_KTB / EB) + i * Tile::RPP < K ? ptr[i] + off : base);
      }
    }
  }
  __device__ __forceinline__ void last_fix(v4i (&reg)[IT], const Last& l) const {
    if constexpr (KC) {
      const int valid = kbytes - (kb + l.ahead * RAGGED_KTB);
      int mask[4];
#pragma unroll
      for (int d = 0; d < 4; d++) mask[d] = valid >= 4 * d + 4 ? -1 : valid <= 4 * d ? 0 : (1 << 8 * (valid - 4 * d)) - 1;
#pragma unroll
      for (int i = 0; i < IT; i++) {
        if (l.shift[i] != 0) reg[i] = chunk_apply<false>(reg[i], chunk_fix(l.shift[i] < 16 ? l.shift[i] : 0, 0, 16));
#pragma unroll
        for (int d = 0; d < 4; d++) reg[i][d] &= mask[d];
      }
    } else {
#pragma unroll
      for (int i = 0; i < IT; i++) {
        reg[i] = chunk_apply<false>(reg[i], edge);
        const bool in = k + l.ahead * (RAGGED_KTB / EB) + i * Tile::RPP < K;
#pragma unroll
        for (int d = 0; d < 4; d++) reg[i][d] = in ? reg[i][d] : 0;
      }
    }
  }
};

// K of a convolution as the kernel walks it: KH runs of KW * Cin bytes, each padded to whole chunks.
template <class P>
static __host__ __device__ __forceinline__ int conv_run(const P& p) { return p.KW * p.Cin; }
template <class P>
static __host__ __device__ __forceinline__ int conv_run_padded(const P& p) { return p.Cin > 0 ? (p.KW * p.Cin + 15) & ~15 : 16; }
// bytes of K as the kernels below walk it
template <bool CONV, int EB, class P>
static __device__ __forceinline__ int walk_bytes(const P& p) {
  if constexpr (CONV) return p.KH * conv_run_padded(p);
  else return p.K * EB;
}

// Position (kh, r) of a K index inside that walk, advanced by `tiles` K tiles at a time without a division.
struct ConvWalk {
  int kh, r, dkh, dr, runp;
  __device__ __forceinline__ void init(int kp, int runp_, int tiles) {
    runp = runp_;
    kh = kp / runp, r = kp - kh * runp;
    dkh = tiles * RAGGED_KTB / runp, dr = tiles * RAGGED_KTB - dkh * runp;
  }
  __device__ __forceinline__ void next() {
    kh += dkh, r += dr;
    if (r >= runp) r -= runp, kh++;
  }
};

// Source of the A operand of a convolution: the NHWC input.
template <int EXT, int THREADS>
struct RaggedImage {
  using Tile = RaggedTile<TypeI8, EXT, THREADS, true>;
  static constexpr int IT = Tile::IT;
  const unsigned char* in;
  int base[IT];     // byte of (image, ih0, iw0, 0), possibly outside the image on its own
  int ih0[IT];      // far outside the image for a row beyond M
  int left[IT];     // bytes of a kernel row that hang over the left edge (<= 0: none)
  int right[IT];    // bytes from the window's first column to the right edge
  int pitch, H, total, KH;
  ConvWalk w;

  // a distance that is only ever compared with positions inside a kernel row (below 2^29 + 16)
  static __device__ __forceinline__ int bounded(int64_t d) {
    const int64_t lim = 1 << 30;
    return (int)(d > lim ? lim : (d < -lim ? -lim : d));
  }
  __device__ __forceinline__ void init(const ConvArgs& p, int m0, int kt0, int t, int tiles = 1) {
    in = (const unsigned char*)p.A;
    pitch = p.W * p.Cin, H = p.H, total = p.a_bytes, KH = p.KH;
    const int cc = t % Tile::CPR, r0 = t / Tile::CPR;
    w.init(kt0 * RAGGED_KTB + cc * 16, conv_run_padded(p), tiles);
#pragma unroll
    for (int i = 0; i < IT; i++) {
      const int m = m0 + r0 + i * Tile::RPP;
      const unsigned mm = m < p.M ? (unsigned)m : 0u;
      const unsigned q = mm / (unsigned)p.OW, img = q / (unsigned)p.OH;
      const int ow = (int)(mm - q * p.OW), oh = (int)(q - img * p.OH);
      const int iw0 = ow * p.stride - p.pad, ih = oh * p.stride - p.pad;
      ih0[i] = m < p.M ? ih : -(1 << 24);
      left[i] = bounded(-(int64_t)iw0 * p.Cin);
      right[i] = bounded((int64_t)(p.W - iw0) * p.Cin);
      base[i] = (((int)img * p.H + ih) * p.W + iw0) * p.Cin;
    }
  }
  __device__ __forceinline__ void load(v4i (&reg)[IT], int (&fix)[IT]) {
#pragma unroll
    for (int i = 0; i < IT; i++) {
      const int ih = ih0[i] + w.kh;
      const int g = base[i] + w.kh * pitch + w.r;
      int lo = left[i] - w.r, hi = right[i] - w.r;  // the bytes of the chunk inside the image row
      const bool in_row = (unsigned)ih < (unsigned)H && w.kh < KH && lo < 16 && hi > 0;
      lo = lo < 0 ? 0 : lo;
      hi = hi > 16 ? 16 : hi;
      int q = g < 0 ? 0 : g;
      q = q > total - 16 ? total - 16 : q;  // the launcher makes sure that there are 16 bytes
      reg[i] = load16_any(in + (unsigned)(in_row ? q : 0));
      fix[i] = in_row ? chunk_fix(g - q, lo, hi) : chunk_fix(0, 0, 0);
    }
    w.next();
  }
};

// Source of the weights of a convolution: a K x N matrix whose rows are picked along the padded walk.
template <int EXT, int THREADS>
struct RaggedWeights {
  using Tile = RaggedTile<TypeI8, EXT, THREADS, false>;
  static constexpr int IT = Tile::IT;
  RaggedMatrix<TypeI8, EXT, THREADS, false> m;  // column handling, guarded loads
  ConvWalk w[IT];
  int64_t ld;
  int run, KH, col;

  __device__ __forceinline__ void init(const ConvArgs& p, int n0, int kt0, int t, int tiles = 1) {
    m.init(p.B, p.ldb, n0, p.N, p.K, 0, t);
    ld = p.ldb, run = conv_run(p), KH = p.KH;
    col = (int)(m.ptr[0] - m.base - (int64_t)(t / Tile::CPR) * ld);  // this thread's column after clamping and shifting
#pragma unroll
    for (int i = 0; i < IT; i++) w[i].init(kt0 * RAGGED_KTB + t / Tile::CPR + i * Tile::RPP, conv_run_padded(p), tiles);
  }
  __device__ __forceinline__ void load(v4i (&reg)[IT], int (&fix)[IT]) {
#pragma unroll
    for (int i = 0; i < IT; i++) {
      const bool in = w[i].kh < KH && w[i].r < run;
      reg[i] = m.guarded(in ? m.base + (int64_t)(w[i].kh * run + w[i].r) * ld + col : m.base, 0, in ? 16 : 0, fix[i]);
      if (in && m.edge != CHUNK_AS_IS) fix[i] = m.edge;
      w[i].next();
    }
  }
};

// AKC / BKC: A (B) is K-contiguous in memory: plain A and B^T are, plain B and A^T are not.  CONV: A is the NHWC input
// and B the weights of a convolution.  R: K tiles in flight in registers.  LONG (products): a row of either operand in
// memory is at least 16 bytes (ragged_long_rows), so whole tiles are loaded without conditions.  Two kernels and not a
// branch: a launch of one tile of short rows fetches its instructions as it goes, and the pipeline's code on the way cost
// it 0.15 us of 3.5 (8 x 8 x 328 4.58 and 4.76, 16 x 912 x 8 3.82 and 4.02).
template <class T, class EPI, int BM, int BN, int WAVES_M, int WAVES_N, bool AKC, bool BKC, bool CONV, bool LONG, int R>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) gemm_ragged_kernel(const std::conditional_t<CONV, ConvArgs, GemmArgs> p) {
  constexpr int THREADS = 64 * WAVES_M * WAVES_N;
  constexpr int EB = T::EB;
  using SA = std::conditional_t<CONV, RaggedImage<BM, THREADS>, RaggedMatrix<T, BM, THREADS, AKC>>;
  using SB = std::conditional_t<CONV, RaggedWeights<BN, THREADS>, RaggedMatrix<T, BN, THREADS, BKC>>;
  using TA = typename SA::Tile;
  using TB = typename SB::Tile;
  constexpr int TM = BM / WAVES_M / 32, TN = BN / WAVES_N / 32, STAGE = TA::BYTES + TB::BYTES;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN, ntiles = tiles_m * tiles_n;
  const int kbytes = walk_bytes<CONV, EB>(p);
  const int nkt_total = (kbytes + RAGGED_KTB - 1) / RAGGED_KTB;
  const int nkt_whole = CONV || !LONG ? 0 : kbytes / RAGGED_KTB;  // tiles before this one lie inside K: unconditional loads
  const unsigned items = (unsigned)ntiles * (unsigned)p.splits;  // (K is cut only where tiles are few)

  for (unsigned item = blockIdx.x; item < items; item += gridDim.x) {
    const int split = p.splits > 1 ? (int)(item / (unsigned)ntiles) : 0;
    int tm, tn;
    tile_coords_mul((int)item - split * ntiles, ntiles, tiles_m, tiles_n, p.band_magic, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int kt0 = p.splits > 1 ? split * p.kt_per_split : 0;
    const int nkt = p.splits > 1 && nkt_total - kt0 > p.kt_per_split ? p.kt_per_split : nkt_total - kt0;

    SA a;
    SB b;
    if constexpr (CONV) {
      a.init(p, m0, kt0, t);
      b.init(p, n0, kt0, t);
    } else {
      a.init(p.A, p.lda, m0, p.M, p.K, kt0, t);
      b.init(p.B, p.ldb, n0, p.N, p.K, kt0, t);
    }
    typename T::accv acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = T::zero();

    auto store = [&](int buf, const v4i (&xa)[SA::IT], const v4i (&xb)[SB::IT]) {
      TA::store(smem + buf * STAGE, t, xa);
      TB::store(smem + buf * STAGE + TA::BYTES, t, xb);
    };
    auto store_fixed = [&](int buf, v4i (&xa)[SA::IT], v4i (&xb)[SB::IT], const int (&fa)[SA::IT], const int (&fb)[SB::IT]) {
#pragma unroll
      for (int i = 0; i < SA::IT; i++) xa[i] = chunk_apply<CONV>(xa[i], fa[i]);
#pragma unroll
      for (int i = 0; i < SB::IT; i++) xb[i] = chunk_apply<false>(xb[i], fb[i]);
      store(buf, xa, xb);
    };
    constexpr int KS = RAGGED_KTB / 32;
    struct Frags {
      v4i a[KS][TM], b[KS][TN];
    };
    auto read = [&](int buf, Frags& f) {
      const unsigned char* As = smem + buf * STAGE;
      const unsigned char* Bs = As + TA::BYTES;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        const int kb = ks * 32 + (lane >> 5) * 16;
#pragma unroll
        for (int i = 0; i < TM; i++) f.a[ks][i] = TA::fragment(As, (wm * TM + i) * 32, kb, lane);
#pragma unroll
        for (int j = 0; j < TN; j++) f.b[ks][j] = TB::fragment(Bs, (wn * TN + j) * 32, kb, lane);
      }
    };
    auto multiply = [&](const Frags& f) {
#pragma unroll
      for (int ks = 0; ks < KS; ks++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) acc[i][j] = EPI::SWAP ? T::mfma(f.b[ks][j], f.a[ks][i], acc[i][j]) : T::mfma(f.a[ks][i], f.b[ks][j], acc[i][j]);
    };
    // The tiles' requests stay in tile order: a wait counts the younger ones, and where a path into a loop has issued
    // them in another order the compiler waits for the worst of both.
    auto in_order = [&]() { asm volatile("" ::: "memory"); };

    if constexpr (CONV) {
      v4i ra[R][SA::IT], rb[R][SB::IT];
      int fa[R][SA::IT], fb[R][SB::IT];
#pragma unroll
      for (int s = 0; s < R; s++) {
        a.load(ra[s], fa[s]);
        b.load(rb[s], fb[s]);
        in_order();
      }
      // Tiles beyond the last are requested like any other (nothing of them is kept): a request that depended on the
      // tile would make every wait below drain all of them.
      for (int kt = 0, buf = 0;;) {
#pragma unroll
        for (int s = 0; s < R; s++) {
          if (kt >= nkt) goto multiplied;
          store_fixed(buf, ra[s], rb[s], fa[s], fb[s]);
          a.load(ra[s], fa[s]);
          b.load(rb[s], fb[s]);
          in_order();
          block_sync();
          Frags f;
          read(buf, f);
          multiply(f);
          buf ^= 1;
          kt++;
        }
      }
    } else if constexpr (!LONG) {
      v4i xa[SA::IT], xb[SB::IT];
      int fa[SA::IT], fb[SB::IT];
      for (int g = 0; g < nkt; g++) {
        a.load_any(xa, fa, g);
        b.load_any(xb, fb, g);
        store_fixed(0, xa, xb, fa, fb);
        block_sync();
        Frags f;
        read(0, f);
        multiply(f);
        block_sync();
      }
    } else {
      // Whole tiles w_0 .. w_(nw - 1) of the slice go through the pipeline: w_k waits in register set k % R, then in LDS
      // buffer k % 2 (R is even).  Trip k reads w_k from LDS, moves w_(k+1) there, requests w_(k+1+R) and multiplies, so
      // the LDS write of one tile runs under the reads and products of another and a tile costs one barrier.  The
      // partial last tile, with its masks, is requested and multiplied ahead of them: no trip then asks what kind of
      // tile it has.
      static_assert(R % 2 == 0, "set and buffer of a trip are constants");
      const int nw = nkt_whole - kt0 < nkt ? (nkt_whole > kt0 ? nkt_whole - kt0 : 0) : nkt;
      v4i ra[R][SA::IT], rb[R][SB::IT];
      auto fetch = [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        a.load_whole(ra[S], a.step);
        b.load_whole(rb[S], b.step);
        in_order();
      };
      auto stage = [&](int buf, auto sc) {  // of a whole tile, only the last chunk of a K-strided row needs its shift
        constexpr int S = decltype(sc)::value;
        if constexpr (!AKC) {
#pragma unroll
          for (int i = 0; i < SA::IT; i++) ra[S][i] = chunk_apply<false>(ra[S][i], a.edge);
        }
        if constexpr (!BKC) {
#pragma unroll
          for (int i = 0; i < SB::IT; i++) rb[S][i] = chunk_apply<false>(rb[S][i], b.edge);
        }
        store(buf, ra[S], rb[S]);
      };
      v4i xa[SA::IT], xb[SB::IT];
      typename SA::Last la;
      typename SB::Last lb;
      if (nw < nkt) {
        a.load_last(xa, la, nw);
        b.load_last(xb, lb, nw);
        in_order();
      }
      int k = 0;
      Frags f;
      // the partial tile, once its requests and those of w_0 .. w_(R - 1) are out
      auto begin = [&](auto refill) {
        if (nw < nkt) {
          a.last_fix(xa, la);
          b.last_fix(xb, lb);
          store(1, xa, xb);
        }
        if (refill.value || nw > 0) stage(0, std::integral_constant<int, 0>{});
        if (refill.value || R < nw) fetch(std::integral_constant<int, 0>{});
        block_sync();
        if (nw < nkt) {
          read(1, f);
          multiply(f);
          block_sync();
        }
      };
      if (nw > 2 * R) {  // requests without conditions from the first to the last steady trip, so that every wait is counted
        for_each_stage(fetch, std::make_integer_sequence<int, R>{});
        begin(std::true_type{});
#pragma unroll 1
        for (; k + 2 * R < nw; k += R) {
          for_each_stage([&](auto sc) {
            constexpr int S = decltype(sc)::value, N = (S + 1) % R;
            read(S & 1, f);
            stage(N & 1, std::integral_constant<int, N>{});
            fetch(std::integral_constant<int, N>{});
            multiply(f);
            block_sync();
          }, std::make_integer_sequence<int, R>{});
        }
      } else {
        for_each_stage([&](auto sc) {
          if (decltype(sc)::value < nw) fetch(sc);
        }, std::make_integer_sequence<int, R>{});
        begin(std::false_type{});
      }
#pragma unroll 1
      while (k < nw) {
        for_each_stage([&](auto sc) {
          constexpr int S = decltype(sc)::value, N = (S + 1) % R;
          if (k < nw) {
            read(S & 1, f);
            if (k + 1 < nw) stage(N & 1, std::integral_constant<int, N>{});
            if (k + 1 + R < nw) fetch(std::integral_constant<int, N>{});
            multiply(f);
            block_sync();
          }
          k++;
        }, std::make_integer_sequence<int, R>{});
      }
    }
  multiplied:
    {
    typename EPI::Pre pre = {};
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) EPI::tile(p, m0 + (wm * TM + i) * 32, n0 + (wn * TN + j) * 32, acc[i][j], lane, split, pre);
    }
    block_sync();  // every wave has read its last fragments before the next item's tiles arrive
  }
}

// Whether a row of either operand in memory is at least 16 bytes (where K is contiguous, that is K).
template <class T, bool AKC, bool BKC>
static bool ragged_long_rows(const GemmParams& p) {
  return (int64_t)(AKC ? p.K : p.M) * T::EB >= 16 && (int64_t)(BKC ? p.K : p.N) * T::EB >= 16;
}
template <class T, class EPI, int BM, int BN, int WAVES_M, int WAVES_N, bool AKC, bool BKC, bool CONV, int R = 2, bool LONG = true>
static hipError_t launch_ragged_tile(const GemmParams& p, hipStream_t stream) {
  if constexpr (!CONV && LONG)
    if (!ragged_long_rows<T, AKC, BKC>(p)) return launch_ragged_tile<T, EPI, BM, BN, WAVES_M, WAVES_N, AKC, BKC, CONV, R, false>(p, stream);
  constexpr int THREADS = 64 * WAVES_M * WAVES_N;
  constexpr int LDS = 2 * (RaggedTile<T, BM, THREADS, AKC>::BYTES + RaggedTile<T, BN, THREADS, BKC>::BYTES);
  auto kern = gemm_ragged_kernel<T, EPI, BM, BN, WAVES_M, WAVES_N, AKC, BKC, CONV, LONG, R>;
  static std::atomic<bool> configured{LDS <= 64 * 1024};
  if (const hipError_t e = allow_dynamic_lds_once(configured, kern, LDS)) return e;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  const int64_t items = (int64_t)tiles_m * tiles_n * p.splits;
  const unsigned grid = (unsigned)(items < (1 << 20) ? items : (1 << 20));  // beyond that the workgroups walk over the items
  const auto args = kernel_args<std::conditional_t<CONV, ConvArgs, GemmArgs>, T>(p, band_magic_of(tiles_m, tiles_n));
  return launch_kernel(kern, dim3(grid), dim3(THREADS), LDS, stream, args);
}

// One output per thread.  For operands of fewer than 16 bytes in all, which have no chunk to load (a matrix of that size has
// K < 16, a convolution input that many values in all, so an output is a handful of products); for products of at most 16
// terms whose rows are short as well, where a chain of sixteen loads is over before a tile's set-up (48 x 3 x 8 4.0 -> 2.6 us,
// 60000 x 8 x 16 7.7 -> 5.2, bf16 3 x 100000 x 5 9.6 -> 3.3); and for a convolution without input channels: its operands
// may be null, no loop below touches them, and the tiled kernel would request its first tiles before it counts them.  (A
// product with K = 0 requests nothing there.)
template <class T, class EPI, bool AKC, bool BKC, bool CONV>
__global__ void __launch_bounds__(256) gemm_tiny_kernel(const std::conditional_t<CONV, ConvArgs, GemmArgs> p) {
  typedef std::conditional_t<T::EB == 1, int, float> val;
  typedef std::conditional_t<T::EB == 1, int8_t, __bf16> elem;
  const elem *A = (const elem*)p.A, *B = (const elem*)p.B;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < (int64_t)p.M * p.N; i += (int64_t)gridDim.x * 256) {
    const int m = (int)(i / p.N), n = (int)(i - (int64_t)m * p.N);
    val s = 0;
    if constexpr (CONV) {
      const int q = m / p.OW, ow = m - q * p.OW, img = q / p.OH, oh = q - img * p.OH;
      const int ih0 = oh * p.stride - p.pad, iw0 = ow * p.stride - p.pad;
      for (int ih = ih0 < 0 ? 0 : ih0; ih < p.H && ih - ih0 < p.KH; ih++)
        for (int iw = iw0 < 0 ? 0 : iw0; iw < p.W && iw - iw0 < p.KW; iw++)
          for (int ci = 0; ci < p.Cin; ci++)
            s += (val)A[((int64_t)(img * p.H + ih) * p.W + iw) * p.Cin + ci] * (val)B[(int64_t)(((ih - ih0) * p.KW + iw - iw0) * p.Cin + ci) * p.ldb + n];
    } else {
      for (int k = 0; k < p.K; k++) s += (val)A[AKC ? (int64_t)m * p.lda + k : (int64_t)k * p.lda + m] * (val)B[BKC ? (int64_t)n * p.ldb + k : (int64_t)k * p.ldb + n];
    }
    EPI::one(p, m, n, s);
  }
}
template <class T, bool AKC, bool BKC, bool CONV>
static bool ragged_tiny(const GemmParams& p) {
  auto bytes = [&](bool kc, int64_t ld, int64_t extent) { return ((kc ? extent - 1 : p.K - 1) * ld + (kc ? p.K : extent)) * T::EB; };
  if (p.K <= 0) return CONV;
  // up to 15 columns (rows) only on small outputs: 8000 x 15 x 16 4.3 -> 4.0 us, 30000 x 15 x 16 4.8 and 8.0
  const int32_t edge = p.M < p.N ? p.M : p.N;
  if (!CONV && p.K <= 16 && (edge <= 8 || (edge < 16 && (int64_t)p.M * p.N <= 1 << 17))) return true;
  return (CONV ? (int64_t)p.a_bytes : bytes(AKC, p.lda, p.M)) < 16 || bytes(BKC, p.ldb, p.N) < 16;
}

// Tile of the ragged kernel: 128 x 128 once such tiles fill half the chip, 64 x 64 otherwise (an edge of less than 192
// wastes too much of the second tile: bf16 130 x 9001 x 301 10.6 us with 128, 9.0 with 64).
static inline int ragged_tile(int32_t M, int32_t N) {
  return M >= 192 && N >= 192 && (int64_t)((M + 127) / 128) * ((N + 127) / 128) >= 128 ? 128 : 64;
}
template <class T, class EPI, bool AKC, bool BKC, bool CONV = false>
static hipError_t launch_ragged(int tile, const GemmParams& p, hipStream_t stream) {
  if constexpr (!std::is_same_v<EPI, EpiloguePartialI32>) {  // (K slices: K is deep)
    if (ragged_tiny<T, AKC, BKC, CONV>(p)) {
      const int64_t blocks = ((int64_t)p.M * p.N + 255) / 256;
      return launch_kernel(gemm_tiny_kernel<T, EPI, AKC, BKC, CONV>, dim3((unsigned)(blocks < (1 << 20) ? blocks : (1 << 20))), dim3(256), 0, stream,
                         (kernel_args<std::conditional_t<CONV, ConvArgs, GemmArgs>, T>(p)));
    }
  }
  if constexpr (!CONV && !std::is_same_v<EPI, EpiloguePartialI32>) {  // (slices: few tiles)
    // Outputs of at most 32 columns on more 64 x 64 tiles than the chip holds at once: 128 x 32 tiles, whose waves all have
    // columns (int8 100000 x 1 x 64 11.7 -> 8.2 us, x 32 x 100 12.5 -> 9.2, 10^6 x 4 x 64 83 -> 49, bf16 100000 x 1 x 64
    // 8.1 -> 6.8; on one round the smaller tile is level or ahead, 30000 x 32 x 100 4.8 and 5.0, 8000 x 8 x 64 4.2 and 4.4).
    if (p.N <= 32 && p.M > 64 * 512) return launch_ragged_tile<T, EPI, 128, 32, 4, 1, AKC, BKC, CONV>(p, stream);
    // 64 x 64 tiles that would leave some compute units with two and others with one become 128 x 64 tiles, one apiece
    // and twice the waves: bf16 1023 x 1537 x 1021 (400 tiles of 64 x 64) 17.6 -> 15.0 us, int8 13.1 -> 10.8, int8
    // 2047 x 800 x 333 6.5 -> 6.3; with one tile to a compute unit anyway the smaller tile wins (int8 1000^3 7.7, 8.1).
    const int64_t tn = (p.N + 63) / 64, tall = (int64_t)((p.M + 127) / 128) * tn;
    if (tile == 64 && tall <= 256 && (int64_t)((p.M + 63) / 64) * tn > 256) return launch_ragged_tile<T, EPI, 128, 64, 4, 2, AKC, BKC, CONV>(p, stream);
  }
  // 128 x 128: sixteen waves of one MFMA tile each for int8, whose products are short beside a trip's other work
  // (2047 x 2045 x 2041 23.2 -> 21.9 us, 1516 x 1764 x 56 6.9 -> 6.1), eight waves of two for bf16 (1500^3 24.0, 26.3)
  constexpr int WAVES_M = T::EB == 1 && !CONV ? 4 : 2;
  return tile >= 128 ? launch_ragged_tile<T, EPI, 128, 128, WAVES_M, 4, AKC, BKC, CONV>(p, stream)
                     : launch_ragged_tile<T, EPI, 64, 64, 2, 2, AKC, BKC, CONV>(p, stream);
}

}  // namespace ac
