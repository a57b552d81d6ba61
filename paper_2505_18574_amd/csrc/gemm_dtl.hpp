// Fast-path tiled MFMA GEMM for gfx950: operands stream global -> LDS directly
// (global_load_lds_dwordx4, no register staging, no ds_write), LDS tiles are
// XOR-swizzled instead of padded, and the K loop is software-pipelined over a
// ring of LDS stages with one workgroup barrier per K tile.
//
// Preconditions (checked by the host launcher; anything else takes the ragged
// kernel in gemm_ragged.hpp): all base pointers 16-byte aligned, row pitches of A
// and B multiples of 16 bytes, K and N multiples of 16 bytes' worth of elements,
// C suitably aligned for vector stores.  M, N, K need not be multiples of the
// tile: out-of-range 16-byte chunks are fetched from a 16-byte block of zeros.
// The DW form of a product asks for multiples of 4 bytes where this says 16
// (dword_operands in common.hpp).
//
// LDS layouts (16-byte slots; a direct-to-LDS wave instruction fills 64
// consecutive slots, the source address of each slot is free):
//   A tile  [BM rows][KTB/16 slots]      slot' = slot ^ ((row / rows-per-256B) & (slots-1))
//   B tile  [KTB/EB k-rows][BN*EB/16]    32-column segments XOR-ed with the k-row (BSwizzle)
// chosen so that the ds_read_b128 of an A fragment (32 rows x 16 B) and the
// transposing ds_read_b64_tr of a B fragment (4 or 8 k-rows x 64 or 32 B) touch
// every LDS bank once.
#pragma once
#include <type_traits>
#include <utility>
#include "gemm_mfma.hpp"
#include "gemm_rules.hpp"

namespace ac {

// 16 bytes of zeros in device memory: the source for chunks outside M, N, K and
// for convolution taps that fall in the padding.
__device__ __attribute__((aligned(16))) const int g_zero16[4] = {0, 0, 0, 0};

// One direct-to-LDS wave instruction: lane i copies 16 bytes from gptr to
// lds_base + 16*i.  Issued through inline assembly so that the compiler does not
// serialise later LDS reads against it; ordering is enforced explicitly with
// wait_vm<N>() + a barrier.  The s_nop is the wait state that an LDS-DMA instruction needs after a scalar write
// of M0 (the compiler pads its own such pairs; it cannot see into the assembly).  It costs nothing measurable.
static __device__ __forceinline__ void load_to_lds16(const void* gptr, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(gptr) : "memory");
}
// Same, with the source given as a wave-uniform base pointer plus a 32-bit byte offset per lane.
static __device__ __forceinline__ void load_to_lds16_so(const void* sbase, unsigned voff, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(voff), "s"(sbase) : "memory");
}
// The same through a buffer descriptor with a 32-bit byte offset per lane: a lane whose offset lies beyond the
// descriptor's size receives zeros (the hardware bounds check), which is how the convolution gather writes its
// padding: no pointer select, no block of zeros.
static __device__ __forceinline__ void buffer_to_lds16(v4i rsrc, unsigned voff, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_base), "v"(voff), "s"(rsrc) : "memory");
}
// 4 bytes per lane: lane i's dword at offset voff (zero beyond the descriptor's size) to lds_base + 4 * i.
static __device__ __forceinline__ void buffer_to_lds4(v4i rsrc, unsigned voff, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds_base), "v"(voff), "s"(rsrc) : "memory");
}
// Descriptor of `bytes` bytes from a wave-uniform address, for raw dword access.
static __device__ __forceinline__ v4i buffer_of(const void* base, unsigned bytes) {
  const uint64_t b = (uint64_t)(uintptr_t)base;
  return (v4i){__builtin_amdgcn_readfirstlane((int)(uint32_t)b), __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)), __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
}
// Workgroup barrier that waits for this wave's LDS traffic only.  __syncthreads() would also drain every
// outstanding global store, which would serialise one tile's epilogue with the next tile's main loop.
static __device__ __forceinline__ void block_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
template <int N>
static __device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// B-tile swizzle.  A transposing read phase touches R k-rows (4 for bf16, 8 for int8) times one
// SEGB-byte segment (64 / 32 bytes: 32 columns).  With RPW rows per 256-byte bank window, XOR-ing the
// segment index with (row / RPW) & MASK spreads those R segments over all 64 banks.
//
// EDGE 16: the fragments of 16 x 16 MFMA tiles take 16 columns at a time, of two of their four 16-byte K chunks in a phase,
// ROWS_PER_CHUNK k-rows apart: the odd chunks exchange the halves of a segment.
template <int EB, int B_ROW, int EDGE = 32>
struct BSwizzle {
  static constexpr int R = EB == 2 ? 4 : 8;
  static constexpr int SEGB = EB == 2 ? 64 : 32;
  static constexpr int SEG_SHIFT = EB == 2 ? 6 : 5;
  static constexpr int SEGS = B_ROW / SEGB;
  static constexpr int RPW = B_ROW >= 256 ? 1 : 256 / B_ROW;
  static constexpr int SPAN = R / RPW < SEGS ? R / RPW : SEGS;
  static constexpr int MASK = SPAN - 1;
  static_assert(SEGS >= 1 && (SEGS & (SEGS - 1)) == 0 && SPAN >= 1, "B tile width must be a power of two of 32-column segments");
  static __device__ __forceinline__ int seg_xor(int row) { return (row / RPW) & MASK; }
  static constexpr int ROWS_PER_CHUNK = 16 / EB;
  static __device__ __forceinline__ int slot_xor(int row) {
    return (seg_xor(row) << (SEG_SHIFT - 4)) ^ (EDGE == 16 ? ((row / ROWS_PER_CHUNK) & 1) << (SEG_SHIFT - 5) : 0);
  }
  // logical 16-byte slot held by physical slot `pslot` of k-row `row` (an involution)
  static __device__ __forceinline__ int slot(int pslot, int row) { return pslot ^ slot_xor(row); }
};

// Swizzled B-fragment reads (see TypeI8/TypeBF16::read_col for the lane roles).
// kb: byte offset of this lane's 16 K-bytes inside the 128-byte K tile; seg: index of the 32-column block.
template <int B_ROW>
static __device__ __forceinline__ v4i dtl_read_col_bf16(const unsigned char* Bs, int kb, int seg, int lane) {
  using S = BSwizzle<2, B_ROW>;
  const int i = lane & 15, g1 = (lane >> 4) & 1;
  const int r = (kb >> 1) + (i >> 2);  // k-row; rows r and r + 4 share one swizzle term
  const unsigned char* p = Bs + r * B_ROW + ((seg ^ S::seg_xor(r)) << 6) + g1 * 32 + 8 * (i & 3);
  v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(AC_LDS(v4s, p));
  v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(AC_LDS(v4s, p + 4 * B_ROW));
  v2i l2 = __builtin_bit_cast(v2i, lo), h2 = __builtin_bit_cast(v2i, hi);
  return (v4i){l2[0], l2[1], h2[0], h2[1]};
}
template <int B_ROW>
static __device__ __forceinline__ v4i dtl_read_col_i8(const unsigned char* Bs, int kb, int seg, int lane) {
  using S = BSwizzle<1, B_ROW>;
  const int i = lane & 15, g1 = (lane >> 4) & 1;
  const int r = kb + (i >> 1);  // k-row; rows r and r + 8 share one swizzle term
  const unsigned char* p = Bs + r * B_ROW + ((seg ^ S::seg_xor(r)) << 5) + g1 * 16 + 8 * (i & 1);
  v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, p));
  v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, p + 8 * B_ROW));
  return (v4i){lo[0], lo[1], hi[0], hi[1]};
}
// Byte offset, inside a B tile, of the first of the two transposing reads of dtl_read_col (the second lies
// HI rows further down), and the fragment read at a given address.
// EDGE 16: seg is the index of the 16-column block.
template <class T, int B_ROW, int EDGE = 32>
static __device__ __forceinline__ int dtl_col_off(int kb, int seg, int lane) {
  using S = BSwizzle<T::EB, B_ROW, EDGE>;
  const int i = lane & 15, g1 = (lane >> 4) & 1;
  if constexpr (EDGE == 16) {
    const int r = T::EB == 2 ? (kb >> 1) + (i >> 2) : kb + (i >> 1);
    return r * B_ROW + (((seg * T::EB) ^ S::slot_xor(r)) << 4) + (T::EB == 2 ? 8 * (i & 3) : 8 * (i & 1));
  } else if constexpr (T::EB == 2) {
    const int r = (kb >> 1) + (i >> 2);
    return r * B_ROW + ((seg ^ S::seg_xor(r)) << 6) + g1 * 32 + 8 * (i & 3);
  } else {
    const int r = kb + (i >> 1);
    return r * B_ROW + ((seg ^ S::seg_xor(r)) << 5) + g1 * 16 + 8 * (i & 1);
  }
}
template <class T, int B_ROW>
static __device__ __forceinline__ v4i dtl_read_col_at(const unsigned char* p) {
  if constexpr (T::EB == 2) {
    v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(AC_LDS(v4s, p));
    v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(AC_LDS(v4s, p + 4 * B_ROW));
    v2i l2 = __builtin_bit_cast(v2i, lo), h2 = __builtin_bit_cast(v2i, hi);
    return (v4i){l2[0], l2[1], h2[0], h2[1]};
  } else {
    v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, p));
    v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32(AC_LDS(v2i, p + 8 * B_ROW));
    return (v4i){lo[0], lo[1], hi[0], hi[1]};
  }
}
template <class T, int B_ROW>
static __device__ __forceinline__ v4i dtl_read_col(const unsigned char* Bs, int kb, int seg, int lane) {
  if constexpr (T::EB == 2) return dtl_read_col_bf16<B_ROW>(Bs, kb, seg, lane);
  else return dtl_read_col_i8<B_ROW>(Bs, kb, seg, lane);
}

// f(integral_constant<0>), f(integral_constant<1>), ...: one call per LDS stage with the stage index a constant.
template <class F, int... I>
static __device__ __forceinline__ void for_each_stage(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

// Bits k = 0 .. n - 1 with 0 <= first + k < extent (kernel rows or columns of a convolution that fall inside the image).
static __device__ __forceinline__ unsigned span_bits(int first, int n, int extent) {
  const int lo = first < 0 ? -first : 0, hi = extent - first < n ? extent - first : n;
  if (hi <= lo) return 0u;
  return (hi >= 32 ? ~0u : (1u << hi) - 1u) & ~((1u << lo) - 1u);
}

// Swizzle term of a row of KTB bytes of K: rows that share a 256-byte bank window get the same.  A 16-byte LDS read serves lanes
// 0-3, 12-15 and 20-27 together, then 4-11, 16-19 and 28-31: with 16 x 16 tiles rows 0-3 and 12-15 of one K chunk and rows 4-11 of
// the next, which the window's number itself puts into the same banks twice where a row has four chunks; its negative does not.
template <int KTB, int EDGE>
static __device__ __forceinline__ int k_row_xor(int row) {
  constexpr int SPR = KTB / 16, RPW = 256 / KTB;
  return (EDGE == 16 && KTB == 64 ? -(row / RPW) : row / RPW) & (SPR - 1);
}

// x as a value of its own: what is computed from it stays where it is written.  (Out of the loop over a workgroup's tiles the
// compiler takes every lane offset that does not change with the tile, some hundred in registers that the tile needs.)
static __device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

template <bool FIRST, class X, class Y>
static __device__ __forceinline__ auto either(const X& x, const Y& y) {
  if constexpr (FIRST) return x;
  else return y;
}

template <class T, int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, int KTB_, int EDGE = 32>
struct DtlGeometry {
  static constexpr int EB = T::EB;
  static constexpr int KSB = EDGE == 16 ? 64 : 32;  // K bytes of an MFMA
  static constexpr int KCH = KSB / 16;              // its 16-byte K chunks: lanes l, l + EDGE, ... hold one each
  using accv = std::conditional_t<EDGE == 16, typename T::acc4, typename T::accv>;
  static constexpr int KTB = KTB_;                // K bytes per A row per tile (64 or 128)
  static constexpr int BK = KTB / EB;             // K elements per tile == k-rows of the B tile
  static constexpr int KSTEPS = KTB / KSB;        // MFMA K-steps per tile
  static constexpr int WAVES = WAVES_M * WAVES_N;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int A_BYTES = BM * KTB;
  static constexpr int A_SPR = KTB / 16;          // slots per A row
  static constexpr int A_ROWS_PER_INSTR = 64 / A_SPR;
  static constexpr int B_ROW = BN * EB;           // bytes per k-row of the B tile
  static constexpr int B_SPR = B_ROW / 16;        // slots per k-row
  static constexpr int B_BYTES = BK * B_ROW;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int LDS_BYTES = STAGES * STAGE;
  static constexpr int A_INSTR = A_BYTES / 1024 / WAVES;  // direct-to-LDS instructions per wave per tile
  static constexpr int B_INSTR = B_BYTES / 1024 / WAVES;
  static constexpr int B_ROWS_PER_INSTR = 64 / B_SPR;
  static constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  static constexpr int TM = WTM / EDGE, TN = WTN / EDGE;
  static_assert(KTB == 64 || KTB == 128, "K tile is 64 or 128 bytes");
  static_assert(A_BYTES % (1024 * WAVES) == 0 && B_BYTES % (1024 * WAVES) == 0, "tile must split into whole wave loads");
  static_assert(B_SPR <= 64 && 64 % B_SPR == 0, "B row must divide a wave load");
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be a multiple of the MFMA's");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
  static __device__ __forceinline__ int a_xor(int row) { return k_row_xor<KTB, EDGE>(row); }
};

// Offsets of the dwords of a last K tile from the tile's origin, for a buffer of DW_REACH bytes (lane_offsets_fit keeps the
// others below that): slot q of the rows from row0 on, byte dw of it; beyond the operand the offset nothing is read at.
constexpr unsigned DW_REACH = 0xfffffff0u, DW_NOTHING = 0xffffffffu;
template <int KTB, int EDGE = 32>  // rows of KTB bytes of K, `rows` and `bytes` of them left
static __device__ __forceinline__ unsigned dword_contiguous(int row0, int q, int dw, int rows, int bytes, int64_t pitch) {
  constexpr int SPR = KTB / 16;
  const int row = row0 + q / SPR, kb = ((q % SPR) ^ k_row_xor<KTB, EDGE>(row)) * 16 + dw;
  return (row < rows) & (kb < bytes) ? (unsigned)row * (unsigned)pitch + (unsigned)kb : DW_NOTHING;
}
template <int EB, int ROW, int EDGE = 32>  // k-rows of ROW bytes, `rows` and `bytes` of them left
static __device__ __forceinline__ unsigned dword_strided(int row0, int q, int dw, int rows, int bytes, int64_t pitch) {
  constexpr int SPR = ROW / 16;
  const int row = row0 + q / SPR, col = BSwizzle<EB, ROW, EDGE>::slot(q % SPR, row) * 16 + dw;
  return (row < rows) & (col < bytes) ? (unsigned)row * (unsigned)pitch + (unsigned)col : DW_NOTHING;
}

// One wave instruction (1 KB of LDS) of a last K tile: 16 bytes per lane at voff, but dword by dword (offset_of(slot, byte)) for
// the one that holds the operand's very last row, `last`, where that ends inside a chunk: no byte behind it is read.
template <class F>
static __device__ __forceinline__ void dw_load(v4i tile, int last, int row0, int rows, int row_bytes, unsigned voff, unsigned lds, int lane, F offset_of) {
  if (row_bytes % 16 != 0 && last >= row0 && last < row0 + rows) {  // wave-uniform
    // a quarter of the instruction's slots at a time: lane l has dword l % 4 of slot 16 s + l / 4
#pragma unroll
    for (int sub = 0; sub < 4; sub++) buffer_to_lds4(tile, offset_of(sub * 16 + (lane >> 2), (lane & 3) * 4), lds + sub * 256);
  } else {
    buffer_to_lds16(tile, voff, lds);
  }
}
// The lane's 16 K-bytes of a fragment, of which `valid` lie inside K; the others are another row's.
static __device__ __forceinline__ v4i dw_mask(v4i f, int valid) {
#pragma unroll
  for (int d = 0; d < 4; d++) f[d] = 4 * d < valid ? f[d] : 0;
  return f;
}

// XCD-aware tile order.  Workgroups are dealt round-robin to the 8 XCDs (each with its own L2), so workgroup b runs on
// XCD b % 8.  Every XCD gets one contiguous run of logical tile ids, and those ids lie in bands of four tile rows, so that
// a run is a compact rectangle sharing A rows and B columns.  No integer divisions: the band size is divided by with a
// multiplier the host supplies, the band height (1 .. 4 tile rows) by a case split.  Two divisions are some sixty
// scalar and vector instructions ahead of a kernel's first load: 0.07 us of a 4 us launch.
static __device__ __forceinline__ void tile_coords_mul(int b, int nblocks, int tiles_m, int tiles_n, unsigned band_magic, int& tm, int& tn) {
  constexpr int XCDS = 8, GROUP_M = 4;
  const int q = nblocks / XCDS, r = nblocks % XCDS;
  const int xcd = b % XCDS, idx = b / XCDS;
  const int id = xcd * q + (xcd < r ? xcd : r) + idx;
  const int group_size = GROUP_M * tiles_n;
  const int group = band_magic ? (int)__umulhi((unsigned)id, band_magic) : id / group_size;
  const int first_m = group * GROUP_M;
  const int gsz = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
  const int in_group = id - group * group_size;
  int qn;
  if (gsz == 4) qn = in_group >> 2;
  else if (gsz == 3) qn = (int)__umulhi((unsigned)in_group, 0x55555556u);  // exact below 2^31
  else if (gsz == 2) qn = in_group >> 1;
  else qn = in_group;
  tm = first_m + (in_group - qn * gsz);
  tn = qn;
}

// Schedules of gemm_dtl_kernel's K loop (each is described at its loop), and the edge of their MFMA tiles.
enum { DTL_ROLLING, DTL_PINGPONG, DTL_INTERLEAVED };
template <int SCHEDULE>
constexpr int dtl_edge = SCHEDULE == DTL_INTERLEAVED ? 16 : 32;

// Whether gemm_dtl_kernel keeps the bias row of its tile in LDS, behind the stages: BN * 4 bytes.
template <class EPI, int BM, int SCHEDULE>
constexpr bool has_bias_lds = (BM >= 256 ? SCHEDULE != DTL_PINGPONG : SCHEDULE == DTL_INTERLEAVED) && std::is_same_v<EPI, EpilogueI8>;

// What an epilogue keeps of its operands over the K loop, a column block of the MFMA's edge.
template <class EPI, int EDGE>
struct epilogue_pre { using type = typename EPI::Pre; };
template <>
struct epilogue_pre<EpilogueI8, 16> { using type = EpilogueI8::Pre16; };

template <int BM, int AMODE>
using dtl_args = std::conditional_t<AMODE == 1, std::conditional_t<(BM >= 256), ConvArgsWide, ConvArgs>, GemmArgs>;

// TA / TB (int8 GEMM): A is given as A^T (K x M, row pitch lda) / B as B^T (N x K, row pitch ldb).
// A transposed operand takes the other operand's role in LDS: A^T is "K-strided" like B (k-rows of BM bytes, the
// B swizzle, fragments through the transposing reads), B^T is "K-contiguous" like A (rows of KTB bytes, the A
// swizzle, 16-byte fragment reads).  The bytes of a tile and the instructions that fill it are the same in either
// role, so only the source offsets, the advance per K tile and the fragment addresses differ.
//
// DW (products): bases, pitches and the contiguous extents are multiples of 4 bytes, not of 16.  A 16-byte load takes any
// dword address, so whole tiles load as before, and a chunk that crosses the end of a row holds the first bytes of the next
// behind it: columns that are never stored or, of a K-contiguous operand, products with k-rows of zeros.  The last K tile reads
// zeros beyond the operands, and its one chunk that could leave a buffer dword by dword; where no zeros face the bytes
// behind K (both operands K-contiguous) or they could be infinite (bf16), A's fragments of that tile are masked.  A contiguous
// extent is at least 16 bytes.
template <class T, class EPI, int BM, int BN, int WAVES_M, int WAVES_N, int AMODE, int STAGES, int KTB_, int SCHEDULE, bool TA = false, bool TB = false, bool DW = false>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) gemm_dtl_kernel(const dtl_args<BM, AMODE> p) {
  constexpr bool PINGPONG = SCHEDULE == DTL_PINGPONG, INTERLEAVED = SCHEDULE == DTL_INTERLEAVED;
  constexpr int EDGE = dtl_edge<SCHEDULE>;
  using G = DtlGeometry<T, BM, BN, WAVES_M, WAVES_N, STAGES, KTB_, EDGE>;
  constexpr int EB = G::EB;
  static_assert(!(TA || TB) || (AMODE == 0 && EB == 1), "transposed operands: int8 GEMM");
  constexpr int AT_ROW = BM * EB, AT_SPR = AT_ROW / 16, AT_RPI = 64 / AT_SPR;  // A^T tile: bytes, slots per k-row, k-rows per instruction
  static_assert(AT_SPR <= 64 && 64 % AT_SPR == 0, "a k-row of A^T must divide a wave load");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const unsigned lds0 = (unsigned)(uintptr_t)AC_LDS(unsigned char, smem);

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int kbytes = p.K * EB, nbytes = p.N * EB;
  const unsigned char* zero = (const unsigned char*)g_zero16;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN, ntiles = tiles_m * tiles_n;
  const int nwork = ntiles * p.splits;

  // Cross-item prefetch (products in ping-pong and interleaved, of 256 x 256 tiles and of 128 x 256): a persistent workgroup requests the first STAGES-1 K tiles of its
  // next output tile before it runs the output stage of the current one, so that the pipeline fill of the next
  // tile and the drain of this tile's stores overlap.  Vector-memory operations of a wave complete in issue order,
  // so the waits of the next tile's first trips name the stores that lie between its loads.
  constexpr bool XPF = (PINGPONG || INTERLEAVED) && AMODE == 0;
  // lower bound of the vector-memory operations one wave issues in the output stage of a FULL tile
  constexpr int EPI_VM = EPI::LDS_STAGED ? G::WTM / 16 * (16 / (64 / (G::WTN / 4))) : G::WTM * G::WTN / 1024;
  constexpr auto vm_count = [](int n) { return n < 63 ? n : 63; };  // vmcnt is a 6-bit counter: naming fewer waits for more

  // The bias of a wave's columns waits in LDS behind the stages, where the tile leaves no registers to hold it over the K
  // loop: 16 to 18 of a wave of the 256 x 128 tiles went to scratch (4784 x 1600 x 2048 24.3 -> 21.8 us, 8192 x 1024 x 1024
  // 14.5 -> 13.6, 3 x 3, 496 -> 304 on 29 images of 27 x 27 47.4 -> 44.7).  The product of a 256 x 256 tile holds them without
  // and is slower with it (5000 x 2560 x 320 12.1 and 13.6); the convolution of that tile spills 19 and still takes registers:
  // its K loop is short more often than long (3 x 3, 64 -> 256 on 64 images of 56 x 56 39.2 us so and 41.7 from LDS, 128 -> 256
  // stride 2 on 192 of 28 x 28 22.1 and 22.8, 5 x 5, 48 -> 224 on 90 of 41 x 41 58.5 and 62.1; 512 -> 512 on 64 of 28 x 28,
  // K = 4608, 121.7 and 118.3; 20 such shapes 1.008 in the mean).  The
  // request is the oldest of its wave, so the K loop's first wait covers it and the barrier behind that publishes it; behind a
  // prefetch (interleaved) it is younger than that item's first tiles, and the last trips, which wait for everything ahead of a
  // barrier, cover it: there are some, since such an item has at least STAGES tiles.  The barrier at the end of the item frees it.
  constexpr bool BIAS_LDS = has_bias_lds<EPI, BM, SCHEDULE>;

  // Stage s: A's tile, then B's, stage after stage; interleaved, all of A's and then all of B's, of 64 KB at most each, which the
  // 16-bit immediate of an LDS read reaches from one lane address an operand.
  constexpr int A_STRIDE = INTERLEAVED ? G::A_BYTES : G::STAGE, B_STRIDE = INTERLEAVED ? G::B_BYTES : G::STAGE;
  constexpr int B_FIRST = INTERLEAVED ? STAGES * G::A_BYTES : G::A_BYTES;
  static_assert(!INTERLEAVED || (STAGES * G::A_BYTES <= 65536 && STAGES * G::B_BYTES <= 65536), "an immediate of 16 bits");

  // ---- item-independent lane roles ---------------------------------------------------------------------
  constexpr int NVAR = G::KTB == 128 ? 2 : 1;
  int a_chunk[NVAR];
#pragma unroll
  for (int v = 0; v < NVAR; v++) a_chunk[v] = (lane % G::A_SPR) ^ G::a_xor(v * G::A_ROWS_PER_INSTR + lane / G::A_SPR);
  const int64_t b_step = (int64_t)G::BK * p.ldb * EB;
  const int64_t a_step_t = (int64_t)G::BK * p.lda * EB;  // A^T: one K tile further down
  v4i a_rsrc = {0, 0, 0, 0};  // the input image
  if constexpr (AMODE == 1) a_rsrc = buffer_of(p.A, (unsigned)p.a_bytes);

  // ---- state of the item whose loads are being issued: per-lane source addressing ------------------------
  // A: wave instruction j (j = wave * A_INSTR + i) fills A_ROWS_PER_INSTR tile rows; lane l -> row
  // j * A_ROWS_PER_INSTR + l / A_SPR, physical slot l % A_SPR, holding logical chunk (l % A_SPR) ^ a_xor(row).
  // The XOR term takes NVAR distinct values per lane as j varies (2 for 128-byte rows, 1 for 64-byte rows).
  // B: wave instruction j fills B_ROWS_PER_INSTR k-rows; lane l -> row j * B_ROWS_PER_INSTR + l / B_SPR,
  // physical slot l % B_SPR.
  // GEMM (AMODE 0): a wave-uniform base pointer per operand that advances by one K tile per issue, plus a
  // constant 32-bit byte offset per lane and instruction.  Rows beyond M and columns beyond N are clamped
  // to valid ones (their products land in accumulators that are never stored); only a partial last K tile
  // needs zeros and takes the slower per-lane pointer path.
  // Convolution (AMODE 1): the row's output pixel gives the byte offset of its window origin in the image
  // (g_base, possibly "negative": only ever used together with an in-range tap) and one bit per kernel row and per
  // kernel column that says whether it falls inside the image (g_rows bit kh, g_cols bit kw; the host keeps KH and KW
  // at most 32).  A load then costs an add, two shifts and two bit operations: a lane whose tap is padding, whose row
  // is beyond M or whose K position is beyond K gets the offset 0xffffffff and the bounds check of the buffer load
  // writes its zeros.  (One bit per tap is one shift less and stops at 32 taps: 7 x 7 kernels then went through the
  // any-alignment gather.  16 -> 112 channels on 22 images of 22 x 22: 16.9 us there, 8.4 here; 224 -> 32 on six of
  // 9 x 9 14.7 and 10.0; 3 x 3 and 5 x 5 kernels 1-5 % faster, the bits being set up without a loop over kernel rows.)
  // The lane's chunk sits at K byte g_kb (the K position of its chunk in the next K tile to be requested), i.e.
  // tap g_kb / Cin, channel g_kb % Cin; both come from two multiply-high divisions per K tile instead of a carried
  // (kh, kw, ci) counter with its loops.
  int split = 0, kt0 = 0, m0 = 0, n0 = 0;
  unsigned a_voff[G::A_INSTR], b_voff[G::B_INSTR];
  int b_krow[G::B_INSTR], a_krow[G::A_INSTR];
  int g_base[G::A_INSTR];
  unsigned g_rows[G::A_INSTR], g_cols[G::A_INSTR];
  unsigned g_kb[NVAR];
  const unsigned char* a_base = nullptr;
  const unsigned char* b_base = nullptr;

  auto setup = [&](int w) {
    const int lane = INTERLEAVED ? opaque(t & 63) : t & 63;
    split = p.splits > 1 ? w / ntiles : 0;
    const int tile = w - split * ntiles;
    kt0 = split * p.kt_per_split;  // first K tile of this slice
    int tm, tn;
    tile_coords_mul(tile, ntiles, tiles_m, tiles_n, p.band_magic, tm, tn);
    m0 = tm * BM, n0 = tn * BN;
#pragma unroll
    for (int i = 0; i < G::A_INSTR; i++) {
      const int row = (wave * G::A_INSTR + i) * G::A_ROWS_PER_INSTR + lane / G::A_SPR;
      const int v = (wave * G::A_INSTR + i) & (NVAR - 1);
      g_base[i] = 0, g_rows[i] = g_cols[i] = 0u, a_voff[i] = 0, a_krow[i] = 0;
      if constexpr (TA) {
        const int krow = (wave * G::A_INSTR + i) * AT_RPI + lane / AT_SPR;
        const int ls = BSwizzle<EB, AT_ROW, EDGE>::slot(lane % AT_SPR, krow);
        a_krow[i] = krow;
        a_voff[i] = (unsigned)krow * (unsigned)(p.lda * EB) + ((m0 + ls * 16) * EB < p.M * EB ? ls * 16 : 0);
      } else if constexpr (AMODE == 0) {
        const int rclamp = m0 + row < p.M ? row : p.M - 1 - m0;
        a_voff[i] = (unsigned)rclamp * (unsigned)(p.lda * EB) + a_chunk[v] * 16;
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
    for (int i = 0; i < G::B_INSTR; i++) {
      if constexpr (TB) {
        const int nrow = (wave * G::B_INSTR + i) * G::A_ROWS_PER_INSTR + lane / G::A_SPR;
        const int rclamp = n0 + nrow < p.N ? nrow : p.N - 1 - n0;
        b_krow[i] = 0;
        b_voff[i] = (unsigned)rclamp * (unsigned)(p.ldb * EB) + a_chunk[(wave * G::B_INSTR + i) & (NVAR - 1)] * 16;
        continue;
      }
      const int row = (wave * G::B_INSTR + i) * G::B_ROWS_PER_INSTR + lane / G::B_SPR;
      const int ls = BSwizzle<EB, G::B_ROW, EDGE>::slot(lane % G::B_SPR, row);
      b_krow[i] = row;
      b_voff[i] = (unsigned)row * (unsigned)(p.ldb * EB) + (n0 * EB + ls * 16 < nbytes ? ls * 16 : 0);
    }
    if constexpr (TA) a_base = (const unsigned char*)p.A + (int64_t)m0 * EB + kt0 * a_step_t;
    else a_base = (const unsigned char*)p.A + (AMODE == 0 ? (int64_t)m0 * p.lda * EB : 0) + (int64_t)kt0 * G::KTB;
    if constexpr (TB) b_base = (const unsigned char*)p.B + (int64_t)n0 * p.ldb * EB + (int64_t)kt0 * G::KTB;
    else b_base = (const unsigned char*)p.B + (int64_t)n0 * EB + kt0 * b_step;
#pragma unroll
    for (int v = 0; v < NVAR; v++) g_kb[v] = (unsigned)(kt0 * G::KTB + a_chunk[v] * 16);
  };

  // Tiles are issued strictly in order 0, 1, 2, ...: the running bases and tap decode rely on it.
  auto issue_loads = [&](int kt_local, int buf) __attribute__((always_inline)) {
    const unsigned As = lds0 + buf * A_STRIDE;
    const unsigned Bs = lds0 + B_FIRST + buf * B_STRIDE;
    const int kt = kt0 + kt_local;
    const int kbase = kt * G::KTB;
    const bool full = kbase + G::KTB <= kbytes - (DW ? 1 : 0);  // wave-uniform; DW: the last tile never is
    if constexpr (DW) {
      if (!full) {
        const v4i a_tile = buffer_of(a_base, DW_REACH), b_tile = buffer_of(b_base, DW_REACH);
        int l = lane;  // opaque, or its offsets are kept in registers from the kernel's start
        asm volatile("" : "+v"(l));
        const int krows = p.K - kt * G::BK;  // k-rows left
#pragma unroll
        for (int i = 0; i < G::A_INSTR; i++) {
          const int j = wave * G::A_INSTR + i, v = (wave * G::A_INSTR + i) & (NVAR - 1);
          if constexpr (TA) {
            dw_load(a_tile, krows - 1, j * AT_RPI, AT_RPI, p.M * EB, a_krow[i] < krows ? a_voff[i] : DW_NOTHING, As + j * 1024, l,
                    [&](int q, int dw) { return dword_strided<EB, AT_ROW, EDGE>(j * AT_RPI, q, dw, krows, p.M * EB - m0 * EB, p.lda * EB); });
          } else {
            const int row = j * G::A_ROWS_PER_INSTR + l / G::A_SPR;
            dw_load(a_tile, p.M - 1 - m0, j * G::A_ROWS_PER_INSTR, G::A_ROWS_PER_INSTR, kbytes,
                    (row < p.M - m0) & (kbase + a_chunk[v] * 16 < kbytes) ? a_voff[i] : DW_NOTHING, As + j * 1024, l,
                    [&](int q, int dw) { return dword_contiguous<G::KTB, EDGE>(j * G::A_ROWS_PER_INSTR, q, dw, p.M - m0, kbytes - kbase, p.lda * EB); });
          }
        }
#pragma unroll
        for (int i = 0; i < G::B_INSTR; i++) {
          const int j = wave * G::B_INSTR + i, v = (wave * G::B_INSTR + i) & (NVAR - 1);
          if constexpr (TB) {
            const int row = j * G::A_ROWS_PER_INSTR + l / G::A_SPR;
            dw_load(b_tile, p.N - 1 - n0, j * G::A_ROWS_PER_INSTR, G::A_ROWS_PER_INSTR, kbytes,
                    (row < p.N - n0) & (kbase + a_chunk[v] * 16 < kbytes) ? b_voff[i] : DW_NOTHING, Bs + j * 1024, l,
                    [&](int q, int dw) { return dword_contiguous<G::KTB, EDGE>(j * G::A_ROWS_PER_INSTR, q, dw, p.N - n0, kbytes - kbase, p.ldb * EB); });
          } else {
            dw_load(b_tile, krows - 1, j * G::B_ROWS_PER_INSTR, G::B_ROWS_PER_INSTR, nbytes, b_krow[i] < krows ? b_voff[i] : DW_NOTHING, Bs + j * 1024, l,
                    [&](int q, int dw) { return dword_strided<EB, G::B_ROW, EDGE>(j * G::B_ROWS_PER_INSTR, q, dw, krows, nbytes - n0 * EB, p.ldb * EB); });
          }
        }
        return;  // the last tile: the running bases are not needed any more
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
        g_kb[v] += G::KTB;
      }
#pragma unroll
      for (int i = 0; i < G::A_INSTR; i++) {
        const int v = (wave * G::A_INSTR + i) & (NVAR - 1);
        const unsigned inside = (g_rows[i] >> g_kh[v]) & (g_cols[i] >> g_kw[v]) & 1u;
        buffer_to_lds16(a_rsrc, ((unsigned)g_base[i] + g_off[v]) | (inside - 1u) | g_dead[v], As + (wave * G::A_INSTR + i) * 1024);
      }
    } else if (full) {
#pragma unroll
      for (int i = 0; i < G::A_INSTR; i++) load_to_lds16_so(a_base, a_voff[i], As + (wave * G::A_INSTR + i) * 1024);
    } else if constexpr (TA) {
#pragma unroll
      for (int i = 0; i < G::A_INSTR; i++) {
        const int k = kt * G::BK + a_krow[i];
        load_to_lds16(k < p.K ? a_base + a_voff[i] : zero, As + (wave * G::A_INSTR + i) * 1024);
      }
    } else {
#pragma unroll
      for (int i = 0; i < G::A_INSTR; i++) {
        const int v = (wave * G::A_INSTR + i) & (NVAR - 1);
        const int kb = kbase + a_chunk[v] * 16;
        load_to_lds16(kb < kbytes ? a_base + a_voff[i] : zero, As + (wave * G::A_INSTR + i) * 1024);
      }
    }
    if (full) {  // every k-row of the tile exists; columns beyond N were clamped when b_voff was set up
#pragma unroll
      for (int i = 0; i < G::B_INSTR; i++) load_to_lds16_so(b_base, b_voff[i], Bs + (wave * G::B_INSTR + i) * 1024);
    } else if constexpr (TB) {
#pragma unroll
      for (int i = 0; i < G::B_INSTR; i++) {
        const int kb = kbase + a_chunk[(wave * G::B_INSTR + i) & (NVAR - 1)] * 16;
        load_to_lds16(kb < kbytes ? b_base + b_voff[i] : zero, Bs + (wave * G::B_INSTR + i) * 1024);
      }
    } else {
#pragma unroll
      for (int i = 0; i < G::B_INSTR; i++) {
        const int k = kt * G::BK + b_krow[i];
        load_to_lds16(k < p.K ? b_base + b_voff[i] : zero, Bs + (wave * G::B_INSTR + i) * 1024);
      }
    }
    a_base += TA ? a_step_t : (int64_t)G::KTB;
    b_base += TB ? (int64_t)G::KTB : b_step;
  };

  typename G::accv acc[G::TM][G::TN];

  // ---- fragments ---------------------------------------------------------------------------------------
  // the lane's A row within an MFMA tile is lane % EDGE, its K chunk lane / EDGE; tile origins are multiples of 16 rows
  // and do not change the swizzle term
  const int a_swz = G::a_xor(lane % EDGE);
  const int a_lane_off = (wm * G::WTM + lane % EDGE) * G::KTB;
  const int b_lane_off_t = (wn * G::WTN + lane % EDGE) * G::KTB;  // B^T: the lane's row of the K-contiguous B tile
  struct Frag {
    v4i a[G::TM], b[G::TN];
  };
  // Of 32 x 32 tiles, the other schedules'.  Written out: through dtl_col_off and with lane / 32 in a variable the register
  // allocator of the A^T products reloaded a lane address from scratch in the K loop (a wait for every request in flight) and kept
  // the arguments of the dword form in lanes of a vector register (256 x 256 tiles, 2 to 4 % of 14 to 41 us).
  auto read_frags = [&](int buf, int ks, Frag& f) {
    const unsigned char* As = smem + buf * A_STRIDE;
    const unsigned char* Bs = smem + B_FIRST + buf * B_STRIDE;
    const int chunk = 2 * ks + (lane >> 5);
#pragma unroll
    for (int i = 0; i < G::TM; i++) {
      if constexpr (TA) f.a[i] = dtl_read_col<T, AT_ROW>(As, chunk * 16, wm * G::TM + i, lane);
      else f.a[i] = *(const v4i*)(As + a_lane_off + i * 32 * G::KTB + ((chunk ^ a_swz) << 4));
    }
#pragma unroll
    for (int j = 0; j < G::TN; j++) {
      if constexpr (TB) f.b[j] = *(const v4i*)(Bs + b_lane_off_t + j * 32 * G::KTB + ((chunk ^ a_swz) << 4));
      else f.b[j] = dtl_read_col<T, G::B_ROW>(Bs, chunk * 16, wn * G::TN + j, lane);
    }
  };
  auto mfma_rows = [&](const Frag& f, int i0, int i1) {  // MFMA row tiles i0 .. i1-1 of one K-step
#pragma unroll
    for (int i = i0; i < i1; i++)
#pragma unroll
      for (int j = 0; j < G::TN; j++) acc[i][j] = EPI::SWAP ? T::mfma(f.b[j], f.a[i], acc[i][j]) : T::mfma(f.a[i], f.b[j], acc[i][j]);
  };
  const int nkt_total = (kbytes + G::KTB - 1) / G::KTB;
  constexpr bool DW_MASK = DW && !TA && (TB || EB == 2);
  auto mask_last = [&](Frag& f, int ks) {
#pragma unroll
    for (int i = 0; i < G::TM; i++) f.a[i] = dw_mask(f.a[i], kbytes - (nkt_total - 1) * G::KTB - (2 * ks + (lane >> 5)) * 16);
  };
  constexpr int PER_TILE = G::A_INSTR + G::B_INSTR;  // outstanding vector-memory ops per tile per wave
  static_assert((STAGES - 1) * PER_TILE <= 63, "vmcnt is a 6-bit counter");
  using SW = BSwizzle<EB, G::B_ROW, EDGE>;
  static_assert(SW::ROWS_PER_CHUNK % SW::RPW == 0 && ((SW::ROWS_PER_CHUNK / SW::RPW) & SW::MASK) == 0, "the B swizzle term must not depend on the K-step");
  constexpr int KS_B = (G::KSB / EB) * G::B_ROW;  // bytes between the B rows of consecutive K-steps
  // a K-contiguous operand needs one lane address per K-step (row tiles are an immediate apart), a K-strided one
  // one per 32-column block (K-steps are an immediate apart)
  constexpr int NAF = TA ? G::TM : G::KSTEPS, NBF = TB ? G::KSTEPS : G::TN;
  constexpr int KS_A = (G::KSB / EB) * AT_ROW;  // A^T: bytes between the rows of consecutive K-steps
  int a_fo[NAF], b_fo[NBF];
#pragma unroll
  for (int x = 0; x < NAF; x++) {
    if constexpr (TA) a_fo[x] = dtl_col_off<T, AT_ROW, EDGE>(lane / EDGE * 16, wm * G::TM + x, lane);
    else a_fo[x] = a_lane_off + (((G::KCH * x + lane / EDGE) ^ a_swz) << 4);
    if constexpr (INTERLEAVED) a_fo[x] = opaque(a_fo[x]);  // or every stage's sum is a register of its own, 64 KB being out of an immediate's reach
  }
#pragma unroll
  for (int x = 0; x < NBF; x++) {
    if constexpr (TB) b_fo[x] = B_FIRST + b_lane_off_t + (((G::KCH * x + lane / EDGE) ^ a_swz) << 4);
    else b_fo[x] = B_FIRST + dtl_col_off<T, G::B_ROW, EDGE>(lane / EDGE * 16, wn * G::TN + x, lane);
    if constexpr (INTERLEAVED) b_fo[x] = opaque(b_fo[x]);
  }
  // The immediate offset of an LDS read has 16 bits: stages that begin 64 KB or more into LDS are read through a
  // second set of lane addresses, 64 KB up (made opaque, or the compiler folds them back into one register per read).
  constexpr bool HI_STAGES = !INTERLEAVED && (STAGES - 1) * G::STAGE >= 65536;
  static_assert((STAGES - 1) * G::STAGE < 2 * 65536, "a third set of lane addresses would be needed");
  int a_fo_hi[NAF], b_fo_hi[NBF];
#pragma unroll
  for (int x = 0; x < NAF; x++) {
    a_fo_hi[x] = a_fo[x] + 65536;
    if constexpr (HI_STAGES) asm volatile("" : "+v"(a_fo_hi[x]));
  }
#pragma unroll
  for (int x = 0; x < NBF; x++) {
    b_fo_hi[x] = b_fo[x] + 65536;
    if constexpr (HI_STAGES) asm volatile("" : "+v"(b_fo_hi[x]));
  }
  // K slices keep the general loops; the convolution gather handles a partial last tile itself
  const int nkt_whole = p.splits > 1 ? 0 : (AMODE == 0 ? (DW ? kbytes - 1 : kbytes) / G::KTB : nkt_total);
  auto issue_whole = [&](auto lbufc) {  // the next tile in order, a whole one, into stage LBUF
    constexpr int LBUF = decltype(lbufc)::value;
#pragma unroll
    for (int i = 0; i < G::A_INSTR; i++) load_to_lds16_so(a_base, a_voff[i], lds0 + LBUF * A_STRIDE + (wave * G::A_INSTR + i) * 1024);
#pragma unroll
    for (int i = 0; i < G::B_INSTR; i++) load_to_lds16_so(b_base, b_voff[i], lds0 + B_FIRST + LBUF * B_STRIDE + (wave * G::B_INSTR + i) * 1024);
    a_base += TA ? a_step_t : (int64_t)G::KTB;
    b_base += TB ? (int64_t)G::KTB : b_step;
  };
  auto issue_whole_rt = [&](int lbuf) {  // the same with the stage as a value (constant after unrolling)
#pragma unroll
    for (int i = 0; i < G::A_INSTR; i++) load_to_lds16_so(a_base, a_voff[i], lds0 + lbuf * A_STRIDE + (wave * G::A_INSTR + i) * 1024);
#pragma unroll
    for (int i = 0; i < G::B_INSTR; i++) load_to_lds16_so(b_base, b_voff[i], lds0 + B_FIRST + lbuf * B_STRIDE + (wave * G::B_INSTR + i) * 1024);
    a_base += TA ? a_step_t : (int64_t)G::KTB;
    b_base += TB ? (int64_t)G::KTB : b_step;
  };
  auto read_frags_at = [&](auto bufc, int ks, Frag& f) {  // read_frags with the stage as a constant
    constexpr int BUF = decltype(bufc)::value;
    constexpr bool HI = BUF * G::STAGE >= 65536;
    constexpr int SOFF = BUF * G::STAGE - (HI ? 65536 : 0);
#pragma unroll
    for (int i = 0; i < G::TM; i++) {
      if constexpr (TA) f.a[i] = dtl_read_col_at<T, AT_ROW>(smem + ((HI ? a_fo_hi[i] : a_fo[i]) + (SOFF + ks * KS_A)));
      else f.a[i] = *(const v4i*)(smem + ((HI ? a_fo_hi[ks] : a_fo[ks]) + (SOFF + i * 32 * G::KTB)));
    }
#pragma unroll
    for (int j = 0; j < G::TN; j++) {
      if constexpr (TB) f.b[j] = *(const v4i*)(smem + ((HI ? b_fo_hi[ks] : b_fo[ks]) + (SOFF + j * 32 * G::KTB)));
      else f.b[j] = dtl_read_col_at<T, G::B_ROW>(smem + ((HI ? b_fo_hi[j] : b_fo[j]) + (SOFF + ks * KS_B)));
    }
  };

  // Persistent workgroups: each takes output tiles blockIdx.x, blockIdx.x + gridDim.x, ...  gridDim.x is a multiple
  // of the number of XCDs (or equals ntiles), so a workgroup's tiles all map to its own XCD in tile_coords_mul().
  // With split-K a work item is (tile, K slice): slice s covers K tiles s * kt_per_split ...
  // The launcher never starts more workgroups than work items, so the first pass needs no test.
  int work = blockIdx.x;
  bool started = false;  // the item's addressing is set up and its first STAGES-1 tiles are requested
  bool pf_stores = false;  // ... and EPI_VM stores of a full tile were issued after those requests
  do {
  if (!started) setup(work);
  const int nkt = p.splits > 1 ? (nkt_total - kt0 < p.kt_per_split ? nkt_total - kt0 : p.kt_per_split) : nkt_total;

#pragma unroll
  for (int i = 0; i < G::TM; i++)
#pragma unroll
    for (int j = 0; j < G::TN; j++) acc[i][j] = typename G::accv{};

  // operands of the output stage that do not depend on the product (bias) are requested before the K loop
  typename epilogue_pre<EPI, EDGE>::type pre[G::TN];
  if constexpr (BIAS_LDS) {
    // no row bias: a buffer of no bytes, which reads as zeros (N is at most 2^29)
    const v4i rsrc = buffer_of(p.bias, p.bias != nullptr && p.bias_ld == 0 ? (unsigned)p.N * 4u : 0u);
    if (wave < BN / 64) buffer_to_lds4(rsrc, (unsigned)(n0 + wave * 64 + lane) * 4u, lds0 + G::LDS_BYTES + wave * 256);
  } else {
#pragma unroll
    for (int j = 0; j < G::TN; j++) EPI::prefetch(p, n0 + wn * G::WTN + j * EDGE, lane, pre[j]);
  }

  if constexpr (INTERLEAVED) {
    // ---- interleaved main loop -------------------------------------------------------------------------
    // Bound by power: what counts is the energy of a product.  A loop of 16 x 16 MFMAs out of registers alone sustains 4100 TOP/s
    // (int8, uniform) and 2080 TFLOP/s (bf16, normal) where one of 32 x 32 does 3500 and 1850: half as many accumulators pass
    // the matrix unit for a product.  Rows of MFMAs alternate their direction, so that one operand stays from each to the next
    // (without, 3830 and 2030).  Four waves of 128 x 128 read two thirds of the fragments that eight of 128 x 64 do.
    // One wave to a SIMD, whose MFMAs leave two or three issue slots each for its other instructions (a 16 x 16 MFMA every 17.3
    // cycles alone, 18.3 with two vector-ALU instructions beside it).  A trip multiplies tile t out of registers and, between
    // the MFMAs, reads the fragments of tile t + 1 (B's into a second set, a row of A's over its own behind the row's last MFMA)
    // and requests a tile.  One barrier a trip, behind its first row of MFMAs: past it tile t + 1 is in LDS for everyone, and
    // everyone has received tile t, whose stage is free.  Eight waves in ping-pong with 16 x 16 MFMAs: 8192^3 int8 432 us, so
    // 418, with the paired requests below 397, its last trips interleaved too 385, with the lane offsets made opaque 380; in
    // ping-pong with 32 x 32 441.  bf16 8192 x 8192 x 4096 461 and 405.
    //
    // Registers are all taken.  The rounds of four trips keep everything in place; around them the allocator moves accumulators and
    // keeps up to 68 bytes a lane in scratch.  The plain int8 form reloads three fragments in its first round behind a prefetch and
    // waits for all requests there, which costs it short K loops (interleaved_rule).  A single copy of the four trips, its first waits
    // chosen at run time or naming no stores, moves 536 to 796 accumulators in every round.
    static_assert(AMODE == 0 && G::KSTEPS == 1 && EDGE == 16 && G::TN % 2 == 0 && STAGES % 2 == 0, "one K-step a tile, two fragment sets in turn");
    constexpr int PPR = G::TN / 2, SLOTS = G::TM * PPR;  // places behind two MFMAs: of a row of tiles, of all
    // A compute unit fetches lines of 128 bytes, two K tiles of a K-contiguous operand: it is requested two tiles at a time, in the
    // odd trips (both stages are free then), a row's second half right behind its first, which the vector L1 still has: 256
    // lines a K tile out of the L2 instead of 384, 5 % of the time.
    constexpr bool PAIR_A = !TA, PAIR_B = TB;
    static_assert(STAGES == 4, "the waits below count the operations of two trips");
    v4i fa[G::TM], fb[2][G::TN];
    if (!started) {
#pragma unroll(DW ? 1 : STAGES)
      for (int s = 0; s < STAGES; s++)
        if (s < nkt) issue_loads(s, s);
    } else {
      issue_whole_rt(STAGES - 1);  // the stage that the output stage of the item before worked in
    }
    // Fragments of the tile in the stage A_STRIDE (B_STRIDE) times its number behind the first.
    auto read_a = [&](int i, int at) {
      if constexpr (TA) fa[i] = dtl_read_col_at<T, AT_ROW>(smem + (a_fo[i] + at));
      else fa[i] = *(const v4i*)(smem + (a_fo[0] + (at + i * EDGE * G::KTB)));
    };
    auto read_b = [&](int j, int at, v4i (&b)[G::TN]) {
      if constexpr (TB) b[j] = *(const v4i*)(smem + (b_fo[0] + (at + j * EDGE * G::KTB)));
      else b[j] = dtl_read_col_at<T, G::B_ROW>(smem + (b_fo[j] + at));
    };
    if (nkt > 0) {
      // tile 0 has landed: the younger tiles (and, after a prefetch, the stores between them) may still be in flight
      if (started && pf_stores) wait_vm<vm_count((STAGES - 1) * PER_TILE + EPI_VM)>();
      else if (STAGES - 1 < nkt) wait_vm<(STAGES - 1) * PER_TILE>();
      else wait_vm<0>();
      block_sync();
#pragma unroll
      for (int j = 0; j < G::TN; j++) read_b(j, 0, fb[0]);
#pragma unroll
      for (int i = 0; i < G::TM; i++) read_a(i, 0);
    } else if constexpr (BIAS_LDS) {
      wait_vm<0>();
      block_sync();
    }
    // The MFMAs of a tile, two by two, with at(place) behind each pair.
    auto places = [&](const v4i (&b)[G::TN], auto at) {
      for_each_stage([&](auto sc) {
        constexpr int S = decltype(sc)::value, i = S / PPR;
#pragma unroll
        for (int e = 0; e < 2; e++) {
          const int jj = 2 * (S % PPR) + e, j = i % 2 == 1 ? G::TN - 1 - jj : jj;
          acc[i][j] = EPI::SWAP ? T::mfma(b[j], fa[i], acc[i][j]) : T::mfma(fa[i], b[j], acc[i][j]);
        }
        __builtin_amdgcn_sched_barrier(0);
        at(sc);
        __builtin_amdgcn_sched_barrier(0);
      }, std::make_integer_sequence<int, SLOTS>{});
    };
    // The row of A that place S reads for the next tile, or -1: a row's fragment is dead behind its last MFMA.
    constexpr auto row_at = [](int s) { return s == SLOTS - 1 ? G::TM - 1 : s >= PPR && s % PPR == 0 ? s / PPR - 1 : -1; };
    // Places behind the barrier that read no row of A, up to S.
    constexpr auto free_before = [](int s) {
      int n = 0;
      for (int x = PPR; x < s; x++) n += !(x == SLOTS - 1 || x % PPR == 0);
      return n;
    };
    constexpr int FREE = SLOTS - PPR - G::TM;
    int kt = 0;
    auto trip = [&](auto bufc, auto extrac) {
      constexpr int BUF = decltype(bufc)::value, NBUF = (BUF + 1) % STAGES;
      constexpr bool ODD = BUF % 2 == 1;
      constexpr int LOADS_A = (PAIR_A ? (ODD ? 2 : 0) : 1) * G::A_INSTR, LOADS_B = (PAIR_B ? (ODD ? 2 : 0) : 1) * G::B_INSTR;
      constexpr int LOADS = LOADS_A + LOADS_B, UNITS = G::TN + LOADS;
      // operations younger than tile kt + 1's: all of two trips' (even); what followed the pairs that it is half of (odd)
      constexpr int YOUNGER = !ODD || (!PAIR_A && !PAIR_B) ? 2 * PER_TILE : PAIR_A ? (PAIR_B ? 0 : 2 * G::B_INSTR) : G::A_INSTR;
      auto load = [&](auto lc) {  // load L of the trip: A's, then B's; of a pair the older tile's, one stage below, first
        constexpr int L = decltype(lc)::value;
        constexpr bool IS_A = L < LOADS_A, PAIR = IS_A ? PAIR_A : PAIR_B;
        constexpr int J = IS_A ? L : L - LOADS_A, I = PAIR ? J / 2 : J;
        constexpr bool OLDER = PAIR && J % 2 == 0;
        if constexpr (IS_A) {
          const unsigned As = lds0 + (BUF - OLDER) * A_STRIDE;
          load_to_lds16_so(PAIR && !OLDER ? a_base + G::KTB : a_base, a_voff[I], As + (wave * G::A_INSTR + I) * 1024);
        } else {
          load_to_lds16_so(PAIR && !OLDER ? b_base + G::KTB : b_base, b_voff[I], lds0 + B_FIRST + (BUF - OLDER) * B_STRIDE + (wave * G::B_INSTR + I) * 1024);
        }
      };
      places(fb[BUF & 1], [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        if constexpr (S == PPR - 1) {
          wait_vm<vm_count(YOUNGER + decltype(extrac)::value)>();
          block_sync();
        }
        if constexpr (row_at(S) >= 0) {
          read_a(row_at(S), NBUF * A_STRIDE);
        } else if constexpr (S >= PPR) {  // B's fragments and the loads, evenly mixed over the free places
          constexpr int Q = free_before(S), U0 = Q * UNITS / FREE, U1 = (Q + 1) * UNITS / FREE;
          for_each_stage([&](auto uc) {
            constexpr int U = U0 + decltype(uc)::value, L = U * LOADS / UNITS;
            if constexpr ((U + 1) * LOADS / UNITS > L) load(std::integral_constant<int, L>{});
            else read_b(U - L, NBUF * B_STRIDE, fb[(BUF & 1) ^ 1]);
          }, std::make_integer_sequence<int, U1 - U0>{});
        }
      });
      a_base += TA ? a_step_t : PAIR_A ? (ODD ? 2 * (int64_t)G::KTB : 0) : (int64_t)G::KTB;
      b_base += TB ? (ODD ? 2 * (int64_t)G::KTB : 0) : b_step;
    };
    const int lim = nkt < nkt_whole ? nkt : nkt_whole;
    {
      // first round after a prefetch across full-tile stores: the loads that trips 0 .. STAGES-3 wait for are
      // older than those stores, so their waits name them instead of draining them
      if (started && pf_stores && kt + 2 * STAGES - 1 < lim) {
        for_each_stage([&](auto bc) {
          if constexpr (decltype(bc)::value < STAGES - 2) trip(bc, std::integral_constant<int, EPI_VM>{});
          else trip(bc, std::integral_constant<int, 0>{});
        }, std::make_integer_sequence<int, STAGES>{});
        kt += STAGES;
      }
    }
    for (; kt + 2 * STAGES - 1 < lim; kt += STAGES)  // tiles kt + STAGES .. kt + 2 STAGES - 1 are whole
      for_each_stage([&](auto bc) { trip(bc, std::integral_constant<int, 0>{}); }, std::make_integer_sequence<int, STAGES>{});
    // The last tiles, up to 2 STAGES - 1 of them, with the stage as a value: what is still to be requested is requested at once,
    // a tile a trip.  When tile kt + 1 has to have landed two younger ones may be in flight at first, then the one that the
    // trip before requested.
    int buf = 0;  // kt is a multiple of STAGES
    auto last_trip = [&](const v4i (&b)[G::TN], v4i (&nb)[G::TN], auto first) {
      const int nbuf = (buf + 1) % STAGES;
      if (kt + STAGES - 1 >= nkt) wait_vm<0>();
      else if (decltype(first)::value && buf == 0) wait_vm<2 * PER_TILE>();
      else wait_vm<PER_TILE>();
      block_sync();
      if (kt + STAGES < nkt) issue_loads(kt + STAGES, buf);
      places(b, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        if constexpr (S < G::TN) read_b(S, nbuf * B_STRIDE, nb);
        if constexpr (row_at(S) >= 0) read_a(row_at(S), nbuf * A_STRIDE);
      });
      buf = nbuf;
      kt++;
    };
    while (kt + 2 < nkt) {
      last_trip(fb[0], fb[1], std::true_type{});
      last_trip(fb[1], fb[0], std::false_type{});
    }
    if (kt + 1 < nkt) {
      last_trip(fb[0], fb[1], std::false_type{});
#pragma unroll
      for (int j = 0; j < G::TN; j++) fb[0][j] = fb[1][j];
    }
    if (nkt > 0) {
      if constexpr (DW_MASK) {
        if (kbytes % 16 != 0 && kt0 + nkt == nkt_total) {
#pragma unroll
          for (int i = 0; i < G::TM; i++) fa[i] = dw_mask(fa[i], kbytes - (nkt_total - 1) * G::KTB - lane / EDGE * 16);
        }
      }
      places(fb[0], [](auto) {});
    }
  } else if constexpr (PINGPONG) {
    // ---- ping-pong main loop ---------------------------------------------------------------------------
    // Eight waves, two per SIMD, in two groups of four (one wave of each group on every SIMD).  A wave
    // alternates between a memory phase (issue its share of the direct-to-LDS loads for a later tile, read
    // all fragments of the current tile into registers) and a compute phase (all MFMAs of that tile), with a
    // workgroup barrier after each phase.  Group 1 is held back by one phase, so at any time one wave per
    // SIMD is feeding the matrix pipe while the other fetches:
    //   phase 2t   : group 0 reads tile t      | group 1 computes tile t-1
    //   phase 2t+1 : group 0 computes tile t   | group 1 reads tile t
    // Tile t sits in stage t % STAGES.  In its memory phase of tile t a wave issues the loads of tile
    // t + STAGES - 1 (into the stage of tile t - 1, whose last reader finished one phase earlier) and waits
    // until its own loads of tile t + 1 have landed; the barrier that ends phase 2t+1 therefore publishes tile
    // t + 1 completely before phase 2t+2 reads it.
    static_assert(!PINGPONG || G::WAVES == 8, "ping-pong needs two waves per SIMD");
    static_assert(!PINGPONG || STAGES >= 3, "ping-pong needs at least three LDS stages");
    const int grp = wave >> 2;
    Frag fr[G::KSTEPS];
    if (!started) {
#pragma unroll(DW ? 1 : STAGES)
      for (int s = 0; s < STAGES - 1; s++)
        if (s < nkt) issue_loads(s, s);
    }
    // tile 0 has landed: the younger tiles (and, after a prefetch, the stores behind them) may still be in flight
    if (XPF && started && pf_stores) wait_vm<(STAGES - 2) * PER_TILE + (XPF ? EPI_VM : 0)>();
    else if (STAGES - 2 < nkt) wait_vm<(STAGES - 2) * PER_TILE>();
    else wait_vm<0>();
    block_sync();                  // tile 0 is visible
    if (grp == 1) block_sync();    // hold group 1 back by one phase
    int buf = 0;
    int kt = 0;
    {
      auto trip = [&](auto bufc, auto extrac) {
        constexpr int BUF = decltype(bufc)::value, LBUF = (BUF + STAGES - 1) % STAGES;
        if constexpr (AMODE == 0) issue_whole(std::integral_constant<int, LBUF>{});
        else issue_loads(kt + BUF + STAGES - 1, LBUF);  // the gather keeps its per-lane addressing; kt is a multiple of STAGES here
#pragma unroll
        for (int ks = 0; ks < G::KSTEPS; ks++) read_frags_at(bufc, ks, fr[ks]);
        wait_vm<(STAGES - 2) * PER_TILE + decltype(extrac)::value>();
        block_sync();
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < G::KSTEPS; ks++) mfma_rows(fr[ks], 0, G::TM);
        __builtin_amdgcn_s_setprio(0);
        block_sync();
      };
      if constexpr (XPF) {
        // first round after a prefetch across full-tile stores: the loads that trips 0 .. STAGES-3 wait for are
        // older than those stores, so their waits name them instead of draining them
        if (started && pf_stores && kt + 2 * STAGES - 2 < nkt_whole && kt + 2 * STAGES - 2 < nkt) {
          for_each_stage([&](auto bc) {
            if constexpr (decltype(bc)::value < STAGES - 2) trip(bc, std::integral_constant<int, EPI_VM>{});
            else trip(bc, std::integral_constant<int, 0>{});
          }, std::make_integer_sequence<int, STAGES>{});
          kt += STAGES;
        }
      }
      // tiles kt + STAGES - 1 .. kt + 2 STAGES - 2, the ones a round of trips requests, are whole
      for (; kt + 2 * STAGES - 2 < nkt_whole && kt + 2 * STAGES - 2 < nkt; kt += STAGES)
        for_each_stage([&](auto bc) { trip(bc, std::integral_constant<int, 0>{}); }, std::make_integer_sequence<int, STAGES>{});
    }
    for (; kt < nkt; kt++) {
      // memory phase
      const int lbuf = buf == 0 ? STAGES - 1 : buf - 1;  // stage of tile kt - 1 == stage of tile kt + STAGES - 1
      if (kt + STAGES - 1 < nkt) issue_loads(kt + STAGES - 1, lbuf);
#pragma unroll
      for (int ks = 0; ks < G::KSTEPS; ks++) read_frags(buf, ks, fr[ks]);
      if (kt + STAGES - 1 < nkt) wait_vm<(STAGES - 2) * PER_TILE>();
      else wait_vm<0>();
      if constexpr (DW_MASK) {
        if (kbytes % 16 != 0 && kt0 + kt == nkt_total - 1) {
#pragma unroll
          for (int ks = 0; ks < G::KSTEPS; ks++) mask_last(fr[ks], ks);
        }
      }
      block_sync();
      // compute phase
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int ks = 0; ks < G::KSTEPS; ks++) mfma_rows(fr[ks], 0, G::TM);
      __builtin_amdgcn_s_setprio(0);
      block_sync();
      buf = buf + 1 == STAGES ? 0 : buf + 1;
    }
    if (grp == 0) block_sync();    // every wave executes the same number of barriers
  } else {
  // Tile t lives in LDS stage t % STAGES.  One fragment set per K-step of a tile stays in registers; as soon
  // as the MFMAs of K-step s of tile kt are issued, the set is refilled with K-step s of tile kt + 1, so an LDS
  // read has the MFMAs of the other K-steps of a tile to land in (with a fragment double buffer per K-step it
  // had one K-step, less than the LDS latency on the small tiles).  One barrier per tile, at the top: past it
  // every wave has received its fragments of tile kt (block_sync waits for the wave's own LDS reads), so the
  // stage of tile kt can take tile kt + STAGES, and tile kt + 1 is visible to everyone.
  Frag fr[G::KSTEPS];
#pragma unroll(DW ? 1 : STAGES)  // one copy of a last tile's code (int8 1000^3 6.9 -> 6.7 us)
  for (int s = 0; s < STAGES; s++)
    if (s < nkt) issue_loads(s, s);
  if (nkt > 0) {
    if (STAGES - 1 < nkt) wait_vm<(STAGES - 1) * PER_TILE>();
    else wait_vm<0>();
    block_sync();
#pragma unroll
    for (int ks = 0; ks < G::KSTEPS; ks++) read_frags(0, ks, fr[ks]);
  } else if constexpr (BIAS_LDS) {
    wait_vm<0>();
    block_sync();
  }
  int buf = 0;
  int kt = 0;
  {
    auto roll = [&](auto bufc) {
      constexpr int BUF = decltype(bufc)::value;
      wait_vm<(STAGES - 2) * PER_TILE>();
      block_sync();
      if constexpr (AMODE == 0) issue_whole(bufc);  // tile kt + STAGES takes the stage that tile kt has just left
      else issue_loads(kt + BUF + STAGES, BUF);
#pragma unroll
      for (int ks = 0; ks < G::KSTEPS; ks++) {
        mfma_rows(fr[ks], 0, G::TM);
        __builtin_amdgcn_sched_barrier(0);
        read_frags_at(std::integral_constant<int, (BUF + 1) % STAGES>{}, ks, fr[ks]);
      }
    };

    const int lim = nkt < nkt_whole ? nkt : nkt_whole;
    for (; kt + 2 * STAGES - 1 < lim; kt += STAGES) {  // tiles kt + STAGES .. kt + 2 STAGES - 1 are whole
      for_each_stage(roll, std::make_integer_sequence<int, STAGES>{});
    }
  }
  for (; kt + 1 < nkt; kt++) {  // every tile but the last
    const int nbuf = buf + 1 == STAGES ? 0 : buf + 1;
    // tile kt + 1 must have landed: only the (STAGES - 2) younger tiles may still be in flight
    if (kt + STAGES - 1 < nkt) wait_vm<(STAGES - 2) * PER_TILE>();
    else wait_vm<0>();
    block_sync();
    if (kt + STAGES < nkt) issue_loads(kt + STAGES, buf);
#pragma unroll
    for (int ks = 0; ks < G::KSTEPS; ks++) {
      mfma_rows(fr[ks], 0, G::TM);
      __builtin_amdgcn_sched_barrier(0);  // keep the refill behind the MFMAs that still read the old fragments
      read_frags(nbuf, ks, fr[ks]);
    }
    buf = nbuf;
  }
  if (nkt > 0) {  // last tile
    if constexpr (DW_MASK) {
      if (kbytes % 16 != 0 && kt0 + nkt == nkt_total) {
#pragma unroll
        for (int ks = 0; ks < G::KSTEPS; ks++) mask_last(fr[ks], ks);
      }
    }
#pragma unroll
    for (int ks = 0; ks < G::KSTEPS; ks++) mfma_rows(fr[ks], 0, G::TM);
  }
  }

  // ---- output stage of the finished item; with XPF the next item's first tiles are requested ahead of it ----
  const int em0 = m0, en0 = n0, esplit = split;
  const int elane = INTERLEAVED ? opaque(lane) : lane;
  const bool efull = em0 + BM <= p.M && en0 + BN <= p.N;  // wave-uniform: no store of this tile is masked
  started = false;
  // What the output stage adds to a lane's four columns in every row, ahead of the next item's tiles, which would be waited for too.
  [[maybe_unused]] const auto add = [&] {
    if constexpr (EPI::LDS_STAGED) return EPI::staged_add(p, en0 + wn * G::WTN + (elane % (G::WTN / 4)) * 4);
    else return 0;
  }();
  if constexpr (XPF) {
    // every item of a launch has the same K range here (no K slices); the fill needs STAGES - 1 whole tiles
    if (work + (int)gridDim.x < nwork && p.splits == 1 && nkt_whole >= (INTERLEAVED ? STAGES : STAGES - 1)) {
      block_sync();  // every wave has read its last fragments: stages 0 .. STAGES-2 can take the next item's tiles
      setup(work + (int)gridDim.x);
#pragma unroll
      for (int s = 0; s < STAGES - 1; s++) issue_whole_rt(s);
      started = true;
      pf_stores = efull;
    }
  }
  if constexpr (EPI::LDS_STAGED) {
    // 4-byte outputs through LDS: the accumulator layout gives a lane one column of many rows, so straight
    // stores are dwords (one 128-byte row segment per half-wave and instruction, 128 instructions per wave for
    // a 64 x 128 wave tile, each about as slow to issue as a 16-byte one).  Every wave instead transposes 16
    // rows of its tile at a time through a private LDS region and stores 16 bytes per lane, whole 128-byte lines
    // per 8 lanes.  With XPF the region lies in the last LDS stage, which the next item does not fill before its
    // first trip: row pitch WTN values with the two half-rows exchanged in rows 4..7 and 12..15, so that the two
    // half-waves, four rows apart, still hit different banks.  Otherwise: row pitch WTN + 8 from the LDS base.
    using SV = typename EPI::StagedValue;
    typedef SV sv4 __attribute__((ext_vector_type(4)));
    // The four lane groups of 16 x 16 tiles are four rows apart: there XPF exchanges the quarters of 64 values by (row / 4) % 4.
    static_assert(XPF || EDGE == 32, "16 x 16 tiles: products, which prefetch");
    constexpr int PITCH = XPF ? G::WTN : G::WTN + 8;
    constexpr auto pcol_of = [](int col, int row) { return !XPF ? col : EDGE == 16 ? col ^ (((row >> 2) & 3) << 4) : col ^ (((row >> 2) & 1) << 5); };
    constexpr int LPR = G::WTN / 4, RPI = 64 / LPR, NI = 16 / RPI;  // lanes per row, rows per instruction, instructions per 16 rows
    static_assert(G::WAVES * 16 * PITCH * 4 <= (XPF ? G::STAGE : G::LDS_BYTES) && 64 % LPR == 0 && 16 % RPI == 0 && sizeof(SV) == 4, "staging region");
    static_assert(!XPF || (G::WTN % 64 == 0), "the half-row exchange needs rows of whole 32-value halves");
    if (!started) block_sync();  // every wave has read its last fragments: the stages are free
    constexpr int RB = 16 * PITCH * 4, AW = G::A_BYTES / RB;  // a wave's bytes; interleaved: waves that work in A's stage, the others in B's
    static_assert(!INTERLEAVED || (AW * RB == G::A_BYTES && (G::WAVES - AW) * RB <= G::B_BYTES), "the last stage, shared out");
    // (As a number of bytes added to smem, which the interleaved loop's is, the region has the ping-pong kernels keep sixteen addresses
    // and write a value at a time: int32 1440 x 9504 x 672 23.6 -> 24.5 us.)
    SV* region = (SV*)(smem + (XPF ? (STAGES - 1) * G::STAGE : 0)) + wave * (16 * PITCH);
    if constexpr (INTERLEAVED) region = (SV*)(smem + (wave < AW ? (STAGES - 1) * A_STRIDE + wave * RB : B_FIRST + (STAGES - 1) * B_STRIDE + (wave - AW) * RB));
    // What is read beside the product is requested for 16 rows at a time, ahead of their way through LDS, and only where there is
    // something to read: a load among the stores, or one that the compiler takes for pending there, is waited for together with
    // every store before it, and with the K tiles that follow.  (Read at each store, us, there / here: int32 without a bias 4952 x
    // 4176 x 2976 91.2 / 82.5, a row 1921 x 416 x 7448 28.0 / 24.6, a matrix 11229 x 2928 x 2464 218 / 152, bf16 with beta 4222 x
    // 6872 x 840 131 / 93; in ping-pong such a matrix 176 and 101.)
    constexpr bool HAS_READS = EPI::STAGED_READS && !INTERLEAVED;  // (launch_dtl_256)
    auto body = [&](auto fullc, auto readsc) {
      constexpr bool READS = decltype(readsc)::value;
#pragma unroll
    for (int i = 0; i < G::TM; i++) {
#pragma unroll
      for (int hf = 0; hf < EDGE / 16; hf++) {
        [[maybe_unused]] sv4 read[NI];
        if constexpr (HAS_READS) {
#pragma unroll
          for (int q = 0; READS && q < NI; q++) {
            const int m = em0 + wm * G::WTM + i * EDGE + hf * 16 + q * RPI + elane / LPR, n = en0 + wn * G::WTN + (elane % LPR) * 4;
            asm volatile("" : "=v"(read[q]));  // any value behind the mask (zeros would be kept in registers over the K loop)
            if (m < p.M && n < p.N) read[q] = EPI::staged_read(p, m, n);
          }
        }
#pragma unroll
        for (int j = 0; j < G::TN; j++)
#pragma unroll
          for (int rr = 0; rr < EDGE / 4; rr++) {
            const int row = (EDGE == 16 ? 0 : 8 * (rr / 4)) + 4 * (elane / EDGE) + rr % 4;
            region[row * PITCH + pcol_of(EDGE * j + elane % EDGE, row)] = EPI::staged_in(p, acc[i][j][hf * 8 + rr]);
          }
        // Other lanes read what this one wrote.  A wave's LDS accesses are in order, but the compiler orders only those of a lane,
        // and moves a write whose own lane does not read it past the reads.
        asm volatile("" ::: "memory");
        if constexpr (READS) {  // received by every lane: what the compiler takes for pending behind a mask it waits for in the next K loop
#pragma unroll
          for (int q = 0; q < NI; q++) asm volatile("" : "+v"(read[q]));
        }
#pragma unroll
        for (int q = 0; q < NI; q++) {
          const int row = q * RPI + elane / LPR, col = (elane % LPR) * 4;
          const sv4 o = *(const sv4*)(region + row * PITCH + pcol_of(col, row));
          const int m = em0 + wm * G::WTM + i * EDGE + hf * 16 + row, n = en0 + wn * G::WTN + col;
          // N is a multiple of 4 on this path: a group of four columns is inside or outside
          if (decltype(fullc)::value || (m < p.M && n < p.N)) EPI::staged_out(p, m, n, o, esplit, either<READS>(read[q], add));
        }
        asm volatile("" ::: "memory");  // ... nor may the next rows be written ahead of the reads
      }
    }
    };
    if constexpr (HAS_READS) {
      if (EPI::staged_reads(p)) body(std::false_type{}, std::true_type{});
      else if (XPF && efull) body(std::true_type{}, std::false_type{});
      else body(std::false_type{}, std::false_type{});
    } else {
      if (XPF && efull) body(std::true_type{}, std::false_type{});
      else body(std::false_type{}, std::false_type{});
    }
  } else if constexpr (BIAS_LDS && EDGE == 16) {
    EpilogueI8::Pre16 bias[G::TN];
#pragma unroll
    for (int j = 0; j < G::TN; j++) bias[j].bias = *(const v4i*)(smem + G::LDS_BYTES + (wn * G::WTN + j * 16 + 4 * (elane >> 4)) * 4);
    EPI::wave_tile(p, em0 + wm * G::WTM, en0 + wn * G::WTN, acc, elane, esplit, bias);
  } else if constexpr (BIAS_LDS) {
    const auto pre_of = [&](int j) {
      asm volatile("" ::: "memory");  // read for each block anew: kept over the blocks they are registers again
      typename EPI::Pre b;
#pragma unroll
      for (int q = 0; q < 4; q++) b.bias[q] = *(const v4i*)(smem + G::LDS_BYTES + (wn * G::WTN + j * 32 + 8 * q + 4 * (elane >> 5)) * 4);
      return b;
    };
    EPI::template wave_blocks<false, G::TM, G::TN>(p, em0 + wm * G::WTM, en0 + wn * G::WTN, [&](int i, int j) -> const typename T::accv& { return acc[i][j]; }, elane, esplit, pre_of);
  } else if constexpr (has_wave_tile<EPI>::value) {
    EPI::wave_tile(p, em0 + wm * G::WTM, en0 + wn * G::WTN, acc, elane, esplit, pre);
  } else {
#pragma unroll
  for (int i = 0; i < G::TM; i++) {
    const int mrow0 = em0 + wm * G::WTM + i * EDGE;
#pragma unroll
    for (int j = 0; j < G::TN; j++) EPI::tile(p, mrow0, en0 + wn * G::WTN + j * EDGE, acc[i][j], elane, esplit, pre[j]);
  }
  }
  block_sync();  // all LDS reads of this tile are done before the next tile refills the LDS stages
  } while ((work += gridDim.x) < nwork);  // tile loop
}

template <class T, class EPI, int BM, int BN, int WAVES_M, int WAVES_N, int AMODE, int STAGES, int KTB_ = 128, int SCHEDULE = DTL_ROLLING, bool TA = false, bool TB = false, bool DW = false>
static hipError_t launch_dtl(const GemmParams& p, hipStream_t stream) {
  using G = DtlGeometry<T, BM, BN, WAVES_M, WAVES_N, STAGES, KTB_, dtl_edge<SCHEDULE>>;
  auto kern = gemm_dtl_kernel<T, EPI, BM, BN, WAVES_M, WAVES_N, AMODE, STAGES, KTB_, SCHEDULE, TA, TB, DW>;
  constexpr int LDS = G::LDS_BYTES + (has_bias_lds<EPI, BM, SCHEDULE> ? BN * 4 : 0);
  static std::atomic<bool> configured{LDS <= 64 * 1024};
  if (const hipError_t e = allow_dynamic_lds_once(configured, kern, LDS)) return e;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  const int ntiles = tiles_m * tiles_n;
  // one persistent workgroup per LDS-limited slot of every compute unit
  constexpr int per_cu = (160 * 1024) / (G::LDS_BYTES > 0 ? G::LDS_BYTES : 1);
  int slots = compute_units() * (per_cu < 1 ? 1 : (per_cu > 8 ? 8 : per_cu));
  slots -= slots % 8;
  if (slots < 8) slots = 8;  // fewer than eight compute units: still a grid, the tile order is a bijection for any size
  const int64_t nwork = (int64_t)ntiles * (p.splits > 1 ? p.splits : 1);
  if (nwork > INT32_MAX) return hipErrorInvalidValue;  // the kernel counts (tile, K slice) items in 32 bits
  const int grid = nwork < slots ? (int)nwork : slots;
  const auto args = kernel_args<dtl_args<BM, AMODE>, T>(p, band_magic_of(tiles_m, tiles_n));
  return launch_kernel(kern, dim3((unsigned)grid), dim3(G::THREADS), LDS, stream, args);
}

// One round of 64 x 128 tiles (gemm_rules.hpp says which calls): three stages of 24 KB, eight waves of 32 x 32.
template <class T, class EPI, int AMODE, bool DW = false, bool TA = false, bool TB = false>
static hipError_t launch_dtl_wide(const GemmParams& p, hipStream_t stream) {
  if constexpr (TA && TB) return launch_dtl<T, EPI, 128, 64, 4, 2, AMODE, 3, 128, DTL_ROLLING, TA, TB, DW>(p, stream);
  else return launch_dtl<T, EPI, 64, 128, 2, 4, AMODE, 3, 128, DTL_ROLLING, TA, TB, DW>(p, stream);
}

// 256 x 256 tiles.  Products whose K loop is long enough run interleaved (interleaved_rule); slices, convolutions, the short ones
// and the output stages that the 16 x 16 tiles do not have stay in ping-pong: int8 shifts and biases (takes16), and those that read a
// matrix beside the product, whose registers the K loop needs (with them bf16 without beta ran 0.96 times as fast as in ping-pong).
template <class T, class EPI, int AMODE, bool TA, bool TB, bool DW>
static hipError_t launch_dtl_256(const GemmParams& p, hipStream_t stream) {
  constexpr bool I8 = std::is_same_v<EPI, EpilogueI8>;
  if constexpr (AMODE == 0 && (I8 || std::is_same_v<EPI, EpilogueRawI32> || std::is_same_v<EPI, EpilogueF32>) && !(TA && !TB)) {
    bool takes;  // the loop's output stage
    if constexpr (I8) takes = EpilogueI8::takes16(p.shift, p.bias, p.bias_ld);
    else takes = !EPI::staged_reads(p);
    if (takes && p.splits <= 1 && interleaved_rule(p.M, p.N, (int64_t)p.K * T::EB, T::EB, I8 ? 1 : 4, TA, TB))
      return launch_dtl<T, EPI, 256, 256, 2, 2, AMODE, 4, 64, DTL_INTERLEAVED, TA, TB, DW>(p, stream);
  }
  return launch_dtl<T, EPI, 256, 256, 2, 4, AMODE, 4, 64, DTL_PINGPONG, TA, TB, DW>(p, stream);
}

// The four direct-to-LDS configurations by tile code.  256: launch_dtl_256, eight waves in ping-pong or four interleaved over four 32 KB
// stages (64 bytes of K per tile; a fifth stage, all of LDS, measured 0.3-1.5 % slower on every large GEMM in ping-pong); 192 (256 x 128),
// 128 and 64: the rolling-refill loop with 128 bytes of K per tile, eight waves of 64 x 64 / 64 x 32 or four waves of
// 32 x 32 (four stages: six and eight were measured slower on every few-tile deep-K shape, 7.9 / 8.3 / 9.3 us on 49 x 2048 x
// 4608: those loops wait on the barrier, not on loads).
template <class T, class EPI, int AMODE, bool DW = false>
static hipError_t launch_dtl_tile(int tile, const GemmParams& p, hipStream_t stream) {
  switch (tile) {
    case 256: return launch_dtl_256<T, EPI, AMODE, false, false, DW>(p, stream);
    case 192: return launch_dtl<T, EPI, 256, 128, 4, 2, AMODE, 3, 128, DTL_ROLLING, false, false, DW>(p, stream);
    case 128: return launch_dtl<T, EPI, 128, 128, 2, 4, AMODE, 3, 128, DTL_ROLLING, false, false, DW>(p, stream);
    default: return launch_dtl<T, EPI, 64, 64, 2, 2, AMODE, 4, 128, DTL_ROLLING, false, false, DW>(p, stream);
  }
}

}  // namespace ac
