// The part of the launch rules that is arithmetic on sizes alone: host code without a HIP header, so that a test can ask
// which kernel a shape takes.
#pragma once
#include <stdint.h>

#include <initializer_list>

namespace ac {

// The plan tables and fits below were measured on the 256 compute units of an MI355X, and the planners are pure host
// arithmetic (the workspace size they imply must not depend on which device happens to be current): they count
// rounds and slots for that chip.  On another compute-unit count the plans stay valid and are merely untuned; the
// launchers size their grids from the device's own count.
constexpr int PLAN_CUS = 256;
struct TiledCost { double c0, per_round, per_round_k; };
struct StationaryCost { double c0, per_k, per_row_tile, per_row_tile_k; };
// time estimate (us) of a tiled code: bm x bn tiles, per_cu workgroups resident per compute unit
inline double tiled_estimate(const TiledCost& c, int bm, int bn, int per_cu, int32_t M, int32_t N, int64_t k128) {
  const int64_t tiles = (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn), slots = PLAN_CUS * per_cu;
  const double rounds = (double)((tiles + slots - 1) / slots);
  return c.c0 + rounds * (c.per_round + c.per_round_k * (double)k128);
}
// ... of a weight-stationary code: every column block of 64 gets the same number of persistent workgroups
inline double stationary_estimate(const StationaryCost& c, int bm, int32_t M, int32_t N, int64_t k128) {
  const int64_t nblk = (N + 63) / 64, tm = (M + bm - 1) / bm;
  int64_t wgs = nblk <= PLAN_CUS ? PLAN_CUS / nblk : 1;
  if (wgs > tm) wgs = tm;
  if (wgs < 1) wgs = 1;
  const double per = (double)((tm + wgs - 1) / wgs), rounds = (double)((wgs * nblk + PLAN_CUS - 1) / PLAN_CUS);
  return c.c0 + rounds * (c.per_k * (double)k128 + c.per_row_tile * per + c.per_row_tile_k * per * (double)k128);
}

// The tile of an int8 product in the range of many_tiles() whose plan the caller did not name: the estimates of
// choose_tile_i8 with the 128 x 256 tile in place of the 256 x 128 one, fitted again to the kernels as they are (least
// absolute deviations on 390 shapes, M 64 .. 8192, N and K 16 .. 8192, operands in the caches, with a bias row; on the
// half held out of a fit the choice is 0.8 % over the best code).  Three stages of 64 bytes of K leave the 128 x 256 tile
// its 72 KB, and rows of C twice as long; the older estimates also put K = 350 .. 800 too low on the weight-stationary
// kernel.  3302 x 1296 x 496 12.3 -> 7.9 us (stationary before), 5676 x 640 x 512 8.7 -> 5.8 (128 x 128 now), 5788 x 960 x
// 192 8.0 -> 6.0, 8192 x 100000 x 80 466 -> 376; over 70 shapes of those ranges outside the fit 0.953 of the time, over 80 of
// 8192 .. 900000 rows or columns 0.966.  Against the kernels and estimates before both, the worst of 114 shapes are 5823 x
// 5696 x 128 19.2 -> 19.9 and 7522 x 3680 x 96 15.2 -> 15.4; the 256 x 128 tile it gave up would still be 2 to 5 % ahead on
// 40811 x 128 x 864 (12.2 and 12.8) and 1776 x 4560 x 5248 (43.0 and 44.0).
// st160_runs, st320_runs: whether the weight-stationary codes may run it (wstat_eligible).
constexpr int TILE_128X256 = 129;  // not a plan's code: this choice alone makes it
inline int choose_product_tile_i8(int32_t M, int32_t N, int32_t K, bool st160_runs, bool st320_runs) {
  static const int codes[4] = {64, 128, TILE_128X256, 256}, bm[4] = {64, 128, 128, 256}, bn[4] = {64, 128, 256, 256}, per_cu[4] = {2, 1, 1, 1};
  static const TiledCost tiled[4] = {{2.377, 0.9053, 0.4796}, {1.999, 1.787, 0.5774}, {0.592, 3.680, 0.8238}, {-0.057, 6.798, 1.2985}};
  static const StationaryCost st160 = {2.447, 0.3235, 0.6542, 0.4560}, st320 = {2.205, 0.4227, 1.0774, 0.6331};
  // from three rounds of the 256 x 256 tile on that tile, as in cheapest_tiled, where three quarters of its edges are used,
  // and before the stationary kernel too (202665 x 464 x 224 89 us there and 74; 276615 x 16 x 240 17.6 and 42.7)
  const int64_t tm = ((int64_t)M + 255) / 256, tn = ((int64_t)N + 255) / 256;
  if (tm * tn >= 768 && 4 * (int64_t)M >= 768 * tm && 4 * (int64_t)N >= 768 * tn) return 256;
  const int64_t k128 = ((int64_t)K + 127) / 128;
  int best = 64;
  double cost = 0.0;
  for (int i = 0; i < 4; i++) {
    const double t = tiled_estimate(tiled[i], bm[i], bn[i], per_cu[i], M, N, k128);
    if (i == 0 || t < cost) cost = t, best = codes[i];
  }
  for (int code : {160, 320}) {
    if (code == 160 ? !st160_runs : !st320_runs) continue;
    const double t = stationary_estimate(code == 160 ? st160 : st320, code == 160 ? 128 : 256, M, N, k128);
    if (t < cost) cost = t, best = code;
  }
  return best;
}

inline int64_t tiles_of(int32_t M, int32_t N, int bm, int bn) { return (((int64_t)M + bm - 1) / bm) * (((int64_t)N + bn - 1) / bn); }

// Tile code for an M x N output when nothing else is known (int32 outputs, convolutions of large kernels): the largest tile
// that still gives most compute units a workgroup (thresholds from exhaustive plan tables on this chip).  A tile much wider or
// taller than the problem wastes most of its MFMAs, so a tile needs 3/4 of its edge in both dimensions.
inline int choose_tile(int32_t M, int32_t N) {
  if (M >= 192 && N >= 192 && tiles_of(M, N, 256, 256) >= 192) return 256;
  if (M >= 192 && N >= 96 && tiles_of(M, N, 256, 128) >= 192) return 192;
  if (M >= 96 && N >= 96 && tiles_of(M, N, 128, 128) >= 128) return 128;
  return 64;
}
// ---- one round of 64 x 128 tiles ---------------------------------------------------------------------------------------
// Outputs of more 64 x 64 tiles than compute units (where some of them get two) of which 64 x 128 tiles make at most one to a
// unit.  What a unit fetches is counted in lines of 128 bytes, one per 1.8 clocks whatever part of it is used (direct-to-LDS
// streams from L2: 147 to 177 KB/us a unit in pieces of 128 bytes, 67 to 78 in pieces of 64), and a k-row of a 64-column int8
// tile is half a line: 64 rows of A and 128 half lines of B are 192 for 64 x 64 outputs, and 192 for 64 x 128.  Eight waves of
// 32 x 32, three stages (four: 1 to 3 % slower below K = 4096; four waves of 32 x 64: 3 to 8).  Measured on 5800 random shapes,
// warm, and 2000 from HBM (before / here, us): 2936 x 384 x 1024 6.3 / 5.5, x 2240 11.5 / 9.0, 1536 x 1024 x 2240 12.9 / 10.1,
// int32 by K 256 .. 8192 1.07 to 1.40 times faster, A^T 1.08 to 1.44, A^T B^T on 128 x 64 tiles 1.06 to 1.3.
inline bool one_round_of_wide_tiles(int32_t M, int32_t N, int bm, int bn) { return tiles_of(M, N, 64, 64) > PLAN_CUS && tiles_of(M, N, bm, bn) <= PLAN_CUS; }
// A product that the others would cut into `splits` pieces (1: none); dw: on dwords.
// Below K = 256 (on dwords 320) the set-up of the wider tile shows (K = 64 3.5 / 3.8); cut products keep their slices beyond
// K = 5000, which are ahead with the weights in HBM (936 x 1200 x 7808 29.0 / 37.3, 436 x 3968 x 3952 28.4 / 19.2).  bf16 rows
// of 64 columns are whole lines: from 640 bytes of K (on dwords 704), on more than 144 tiles (129 of them 16.7 / 18.7 from HBM at
// 2717 x 384 x 2240), and uncut only, so that the sums keep their order.
inline bool wide_product_rule(int32_t M, int32_t N, int64_t kbytes, int eb, bool dw, int splits) {
  if (!one_round_of_wide_tiles(M, N, 64, 128)) return false;
  if (eb == 2) return splits <= 1 && kbytes >= (dw ? 704 : 640) && tiles_of(M, N, 64, 128) > 144;
  return kbytes >= (dw ? 320 : 256) && (splits <= 1 || kbytes <= 5000);
}
// An int8 product with transposed operands, never cut.  B^T has whole lines on either tile; its products on dwords stay (1.00
// in the mean), and those of A^T B^T beyond K = 3000 (0.92 to 1.01).  A^T B^T is wide in M.
inline bool wide_trans_rule(int32_t M, int32_t N, int32_t K, bool trans_a, bool trans_b, bool dw) {
  if (!one_round_of_wide_tiles(M, N, trans_a && trans_b ? 128 : 64, trans_a && trans_b ? 64 : 128)) return false;
  if (!trans_a) return !dw && K >= 640;
  return K >= 256 && !(trans_b && dw && K > 3000);
}
// ---- at most 32 columns on more rows than the shared tiles take: 128 x 32 tiles (gemm_i8.hip, launch_narrow) --------------
// Rows that are read once, beside the weight-stationary kernel, which keeps more loads in flight where the rows are many (us there /
// here): 137103 x 32 x 128 8.7 / 7.4, 282133 x 32 x 208 16.5 / 14.0, 290715 x 32 x 544 38.4 / 38.0, but 753035 x 16 x 128 24.3 / 27.9,
// 574609 x 32 x 352 47.3 / 50.5, 1837930 x 16 x 176 73.5 / 81.9; a short K earlier: 96366 x 32 x 16 5.3 / 4.7 and 401408 x 16 x 80 13.5 /
// 14.1; 1 x 1 stride 2, 48 -> 16 on 100719 pixels 7.4 / 7.0, on 164836 9.3 / 9.8, on 1052025 34.0 / 45.5; 2 x 2 stride 2, 176 -> 32 on
// 960000 142 / 162.  Beside the 64 x 64 tile as well: 2 x 2 stride 2, 352 -> 16 on 349856 pixels 107 / 118.
inline bool narrow_rows_rule(int32_t M, int32_t K) { return M <= 512 * PLAN_CUS || (K >= 128 && M <= 1152 * PLAN_CUS); }
// Such rows beside the 64 x 64 tile: a deep K is all waiting for them, and the compute unit with the most counts.  Where tiles of 64
// rows deal them more evenly those stay (48529 x 32 x 2192, 256 rows and 192, 24.8 / 27.3, 36048 x 32 x 2960 28.9 / 33.8, 70643 x 16 x
// 2288, 384 and 320, 37.6 / 40.7, 3 x 3 stride 3, 368 -> 16 on 35525 pixels 30.6 / 36.8; 38235 x 32 x 160 4.4 / 4.0, 40867 x 16 x 1088
// 12.1 / 10.7, 87408 x 32 x 2304, 384 and 384, 42.7 / 40.4).
inline int64_t busiest_unit_rows(int32_t M, int bm) { return (((int64_t)M + bm - 1) / bm + PLAN_CUS - 1) / PLAN_CUS * bm; }
inline bool narrow_rows_even(int32_t M, int32_t K) { return K < 1100 || 20 * busiest_unit_rows(M, 128) <= 23 * busiest_unit_rows(M, 64); }
// An int8 product, against the stationary kernel or the 64 x 64 tile: 50176 x 32 x 1024 11.6 / 9.8, 200704 x 32 x 256 13.3 / 11.5, 41876 x
// 32 x 208 5.0 / 4.1, 27225 x 16 x 32 3.6 / 3.4.
inline bool narrow_product_rule(int32_t M, int32_t N, int32_t K) { return N <= 32 && M > 64 * PLAN_CUS && narrow_rows_rule(M, K) && narrow_rows_even(M, K); }
// A convolution of at most 64 output channels on more than one 64 x 64 tile per compute unit: that tile, uncut, or up to 32
// channels the 128 x 32 one (narrow_conv_tile).  The planner's estimates, made for products, take wider tiles or K slices
// there, which compute or store columns that do not exist (7 x 7, 224 -> 32 channels on 43 images of 25 x 25 53 -> 34 us, 5 x 5 stride 2, 496 -> 48 on 42 of
// 55 x 55 101 -> 77; level on the shapes where they agree).  Where they take the weight-stationary kernel (`stationary`) they are
// right as long as K is short, and a single tap, a plain product but for its rows, always is (1 x 1 stride 2, 64 -> 48 on 64
// images of 56 x 56 6.6 us there and 8.8 on the tile); its gather loses from K = 800 on where the columns are whole 32s (from
// 400 with more than nine taps), from 1200 on otherwise (3 x 3 stride 2, 96 -> 64 on 76800 pixels 20.8 and 14.3, 5 x 5 stride 2,
// 16 -> 64 on 39546 10.5 and 7.8; 144 -> 64 on 285696, K = 576, 32.9 and 35.4).  Sixty-four columns fill half of a wide tile, which is
// the better one for K beyond 32768 (5 x 5, 1968 -> 64 on 51840 pixels 378 and 410, 1520 -> 64 339 and 350; 1056 -> 64 on 39546, K =
// 26400, 182 and 147).
// The 128 x 32 tile is ahead of the 64 x 64 one on all of 60 such convolutions, 1.2 times in the mean (3 x 3, 512 -> 32 on 50176 pixels
// 29.8 -> 19.2 us, 5 x 5, 112 -> 16 on 290238 83.6 -> 47.4, 7 x 7, 128 -> 32 on 145119 85 -> 57), and of the weight-stationary kernel
// wherever windows overlap (3 x 3, 48 -> 32 on 139240 pixels 18.6 -> 10.5, 80 -> 16 on 40768 10.6 -> 6.5; 5 x 5 stride 2, 48 -> 32 on 1802493
// 295 -> 200); where they do not, rows are read once, as a product's are.
inline bool narrow_conv_tile(int32_t M, int32_t N, int32_t K, int32_t taps, int32_t stride) {
  return N <= 32 && (taps > (int64_t)stride * stride || (narrow_rows_rule(M, K) && narrow_rows_even(M, K)));
}
inline bool narrow_conv_rule(int32_t M, int32_t N, int32_t K, int32_t taps, int32_t stride, bool one_wave, bool stationary) {
  if (N > 64 || M <= 64 * PLAN_CUS || one_wave || (N > 48 && K > 32768)) return false;
  return !stationary || narrow_conv_tile(M, N, K, taps, stride) || K >= (N % 32 != 0 ? 1200 : taps > 9 ? 400 : 800);
}
// Beside the patch kernel, few of whose pixels meet at a stride: 5 x 5 stride 2, 32 -> 32 on 89 images of 59 x 59 12.6 -> 9.5 us, 3 x 3
// stride 2, 64 -> 16 on 83 of 64 x 64 12.9 -> 10.1, 2 x 2 stride 2, 32 -> 16 on 1441557 pixels 113 -> 63; at stride 1 it is ahead on
// most (64 -> 32 on 94 of 55 x 55 16.0 and 18.6).
inline bool narrow_conv_instead_of_patch(int32_t M, int32_t N, int32_t stride) { return stride > 1 && N <= 32 && M > 64 * PLAN_CUS; }
// A convolution of `taps` kernel positions over `bytes` of input and weights.  Its gather issues an address per 16 bytes, and two
// workgroups of 64 x 64 to a unit cover that better than one where the lines come from near by: kernels whose positions
// overlap more than ten times on 2.5 MB and less stay (7 x 7, 64 -> 128 on 11264 pixels 12.1 / 12.9).  336 -> 112, 3 x 3 stride 2 on
// 9522 pixels 16.0 / 12.5, 416 -> 336 on 3872 20.0 / 15.3, 128 -> 272 on 61 images of 8 x 8, taken from the patch kernel, 12.9 / 7.1.
// K beyond 8192 stays with its slices (496 -> 240 on 5746 pixels, K = 24304, 56.8 / 70.7).
// Up to K = 640 in whole 64s the plan here is the kernel of one wave to a tile, which keeps those it walks in 64 bytes of K, ten waves to a
// unit, where windows overlap on up to some six tiles a unit, at a stride four (64 -> 160, 3 x 3 on 6348 pixels 4.9 / 5.7, 64 -> 288 on 5000,
// 1413 tiles, 5.1 / 5.8, 80 -> 176, 2 x 2 on 5832 4.2 / 4.9; stride 2, 64 -> 144 on 6156, 965 tiles, 5.0 / 5.7; given up: 64 -> 368 on 4050, 1524
// tiles, 7.1 / 5.9, stride 2, 64 -> 416 on 3200, 1300 tiles, 7.1 / 5.9, 64 -> 352 on 5239 9.0 / 5.9).  On its 128 bytes, six waves to a unit, it is level to 1.5 times slower (128 -> 384, 2 x 2 on 4225 7.4 / 5.3, K = 640 1.25 in the mean), without overlap
// 1.0 to 1.8 (1 x 1 stride 2, 576 -> 112 on 13068 8.5 / 5.9); other K there never were its (1 x 1 stride 2, 544 -> 192 6.1 / 5.7).
inline bool wide_conv_rule(int32_t M, int32_t N, int32_t K, int32_t taps, int32_t stride, int64_t bytes) {
  if (!one_round_of_wide_tiles(M, N, 64, 128) || K < 256 || K > 8192) return false;
  if (K % 128 == 64 && K <= 576 && taps > (int64_t)stride * stride && tiles_of(M, N, 32, 32) <= (stride == 1 ? 1500 : 1024)) return false;
  return taps <= 10 * (int64_t)stride * stride || bytes > 2500000;
}

// ---- gemm_kgroup.hpp: which calls its kernels take from the others ------------------------------------------------------
// A product (or, `conv`, a convolution as its implicit product) and how the other kernels would run it.
struct KGroupCall {
  int32_t M, N, K;
  int eb;  // bytes of an element
  bool conv;
  bool a_along_k, b_along_k;  // the operand's rows run along K in memory (a plain A and a B^T do)
  int64_t b_pitch;            // bytes
  int splits;                 // pieces that the others would cut K into over workgroups (1: none)
  bool workspace;             // ... through a workspace; without one bf16 slices meet in atomics
  int32_t Cin;                // conv
  bool raw = false;           // int32 outputs, whose other tile is the 64 x 64 one whatever K
};

// The kernel on direct-to-LDS operands.  On 430 random shapes per form, warm and from HBM, in us (there / here):
//   up to 256 tiles, a round of eight-wave workgroups, it is ahead for every K the others do not cut (128 x 1024 x 3072
//   without a workspace 8.9 / 5.2, 16 x 2048 x 2304 6.6 / 4.1, int32 128 x 128 x 2048 5.9 / 3.8, bf16 256 x 256 x 1024 7.0 /
//   3.6, 3 x 3, 256 -> 256 on one 14 x 14 image 8.3 / 4.4, 256 x 64 x 128 one wave to a tile 2.8 / 2.7);
//   up to 512 tiles, two rounds of four waves each, only where K is short (2350 x 256 x 176 4.4 / 3.4, 608 x 576 x 256
//   3.5 / 3.5, 224 x 1920 x 624 4.3 / 4.5), shorter where no operand's rows run along it (A^T 64 x 5584 x 336 3.8 / 3.7, 1328 x
//   352 x 448 4.0 / 4.6), longer where both operands' do (B^T 256 x 1072 x 1280 5.8 / 4.0);
//   longer for int32 outputs (7468 x 44 x 640 5.3 / 4.0, 700 x 532 x 904 6.2 / 5.3, from HBM 8.0 / 6.9; 4672 x 64 x 896 5.1 / 3.7; given
//   back: 560 x 784 x 1024 5.1 / 5.6);
//   against the kernel of one wave to a tile up to 256 tiles, but for a few tiles of one K tile, where one wave has all the work
//   (57 x 64 x 64 2.5 / 2.65, 30 x 64 x 256 2.7 / 2.5, 100 x 256 x 64 3.0 / 2.7).
// Where the others would cut K, slices have more of B in flight, and what decides is where the weights come from: from HBM a
// compute unit's whole share of B in 32-byte pieces is the limit.  The line lies where two shapes of 430 are more than a tenth
// behind from HBM, and none is when they come from the last-level cache (slices / here, warm and from HBM: 344 x 480 x
// 3136 9.0 / 5.9 and 11.5 / 9.1, 58 x 512 x 2144 7.1 / 3.9 and 9.7 / 8.3; given back: 16 x 4096 x 4096 8.6 / 6.0 and 11.8 /
// 15.7, 26 x 896 x 3520 7.7 / 4.7 and 9.8 / 11.6, bf16 16 x 896 x 2432 5.8 / 4.8 and 7.2 / 9.8, 3 x 3, 512 -> 512 on a 7 x 7
// image 7.3 / 5.7 and 9.1 / 13.1).  More tiles move it up (the slices' sums are more), eight slices down (they share B
// further), and rows of B a multiple of 2 KB apart (bf16: 1 KB) are left to the slices (16 x 2048 x 2048 from HBM 8.3 / 9.4,
// 16 x 2064 x 2048 9.2 / 7.9).  Where B is narrow its lines are used whole (1400 x 32 x 4352 8.6 / 4.4 and 10.1 / 8.8).
// Convolutions whose weights are few, up to 128 columns, come from the slices to a K that grows with the tiles: their images,
// not their weights, are what a compute unit streams, and each pixel's chunks serve all columns of a tile.  (Slices / here, warm and
// from HBM: 304 -> 16, 5 x 5 on 4232 pixels 13.1 / 6.7 and 14.0 / 8.1; 256 -> 32, 7 x 7 on 5618 23.3 / 8.8 and 22.6 / 11.7; 240 -> 48,
// 5 x 5 on 700 8.0 / 5.9 and 8.3 / 6.6; 256 -> 80 on 1980 13.2 / 7.6 and 13.7 / 11.1.)  The fewest tiles keep the line of the products
// (100 x 64 x 5040); left to the slices 320 -> 80 on 512 8.9 / 6.8 and 9.7 / 12.4, 480 -> 32 on 450, K = 12000, 8.2 / 8.3 and 9.2 / 14.3.
// Of 130 in the upper half of the line none is behind warm (1.27 times faster in the mean); from HBM 1.08, and 19 are more than a
// twentieth behind, up to a quarter: many channels at a stride under 96 and more columns (544 -> 112, 3 x 3 stride 2 on 324
// pixels 7.8 / 6.2 and 9.0 / 11.7, 640 -> 128 on 825 9.6 / 9.4 and 11.0 / 13.9).
// Two rounds of four waves (t > 256) are ahead of the 64 x 64 tiles and their slices on these as well (448 -> 32, 3 x 3 on 11264 pixels
// 12.6 / 7.7 and 12.7 / 9.9, 112 -> 48, 5 x 5 stride 1 on 5476, K = 6000, 13.9 / 9.9 and 14.4 / 11.9; given back: 432 -> 64, K = 10800, 18.8 /
// 17.6 and 18.2 / 21.5) while the weights, which every second tile streams again, are some 600 KB (208 -> 112, 5 x 5 on 3211 14.8 / 13.0 and
// 16.3 / 14.7, 192 -> 96 on 4056 15.2 / 11.0; 272 -> 128, 5 x 5 stride 2 on 2448 14.1 / 18.6 and 17.1 / 21.1, 816 -> 128, 3 x 3 on 3072 15.0 /
// 20.9, 144 -> 112, 7 x 7 stride 2 on 3200 14.5 / 17.1) and, of more than 80 columns, some units have one tile left (144 -> 128, 5 x 5
// stride 2 on 3920, 492 tiles, 11.7 / 13.1).  With up to 400 columns as long as K is some 4000 on up to 384 tiles (144 ->
// 240 on 1372 13.3 / 10.7 and 14.6 / 12.5, 368 -> 160 on 2124 14.5 / 10.4 and 15.3 / 13.3; beyond, 288 -> 448 on 960, K = 2592, 8.9 / 9.6, 352 ->
// 464, 3 x 3 stride 2 on 722 10.8 / 12.9, 320 -> 512 on 588 9.9 / 11.3).
inline int64_t kgroup_cut_conv_limit(int row, int64_t t) {
  if (row <= 16) return t <= 81 ? 9600 + 128 * t : 20000;
  if (row <= 32) return t <= 4 ? 9600 : 8800 + 40 * t;
  if (row <= 64) return t <= 8 ? 4800 : 6400 + 22 * t;
  return 3900 + 28 * t;
}
inline int64_t kgroup_two_rounds_conv_limit(int32_t N, int64_t t) {
  if (N <= 128) return N > 80 && t > 480 ? 2400 : N <= 76 ? 8000 : 615000 / N;
  return N <= 400 && t <= 384 ? 4000 : 2400;
}
inline bool kgroup_rule(const KGroupCall& c) {
  const int64_t t = tiles_of(c.M, c.N, 32, 32), kbytes = (int64_t)c.K * c.eb, row = (int64_t)c.N * c.eb;
  if (c.K < 16 || c.N < 1) return false;
  if (t > 256) return t <= 512 && kbytes <= (c.conv ? kgroup_two_rounds_conv_limit(c.N, t) : c.raw ? (c.N <= 64 ? 1408 : 960) : c.b_along_k || c.eb == 2 ? 1280 : c.a_along_k ? 608 : 352);
  if (c.splits <= 1) return true;
  if (!c.workspace) return kbytes <= (row <= 64 ? 7168 : 5120);  // atomics, whose sums differ from run to run
  if (c.conv && row <= 128) return kbytes <= kgroup_cut_conv_limit((int)row, t);
  if (row <= 64) return kbytes <= (t <= 2 ? 7168 : 4480);
  if (c.splits >= 8) return false;
  if (c.conv) return kbytes <= 7200 && kbytes <= 3392 + 10 * t;
  if (c.b_pitch % (2048 / c.eb) == 0) return false;
  return c.eb == 2 ? kbytes <= 5120 && kbytes <= 3712 + 8 * t : kbytes <= 4096 && kbytes <= 2912 + 8 * t;
}

inline bool kgroup_instead_of_one_wave(int32_t M, int32_t N, int32_t K) {
  const int64_t t = tiles_of(M, N, 32, 32);
  return t <= 256 && (K > 64 || t > 16);
}

// The same question for operands of any alignment, whose other kernels cost a K tile 0.26 us.  On 200 random shapes (there /
// here): up to 256 tiles ahead from K of 16 bytes on (91 x 54 x 19 4.3 / 3.7 us, int32 18 x 35 x 32 4.5 / 3.3, 106 x 360 x
// 1476 with A^T 10.1 / 5.9, 872 x 29 x 1397 8.9 / 5.9, bf16 478 x 485 x 536 7.2 / 5.5, 5 x 5, 59 -> 57 on one 13 x 13 image 15.7 /
// 8.0), but for convolutions of K below 200, which conv_image.hpp does as well (64 x 22 x 153 4.9 / 5.1), up to 320 or 800 where
// its loads are whole dwords or chunks and the columns few (3 x 3, 32 -> 6 on 6728 pixels 4.5 / 5.2, 64 -> 20 on 300 5.6 / 6.0);
// and for cut products on the line above, drawn lower here (slices / here, warm and from HBM: 25 x 1000 x 2557 8.2 / 5.7
// and 10.5 / 10.5, 20 x 485 x 3244 8.8 / 8.2 and 11.0 / 12.9, 317 x 262 x 3123 9.7 / 10.6 and 11.9 / 12.5).
// Up to 448 tiles with half the waves, as long as two rounds of them keep up with the wider tiles there (195 x 1599 x 233 5.1 /
// 4.3, 621 x 509 x 2394 11.7 / 13.9, A^T 361 x 1101 x 1542 11.1 / 12.7, B^T 465 x 733 x 3258 11.2 / 10.5, bf16 1383 x 293 x
// 6769 41.5 / 44.6), for convolutions from K = 1200 on (3 x 3, 54 -> 54 on 6075 pixels 15.0 / 12.0, 12943 x 25 x 925 9.7 / 9.7),
// 2400 with whole chunks (5 x 5, 48 -> 198 on 1600 9.2 / 11.9), which their slices beat where the columns are many or K is deep (5 x
// 5, 226 -> 126 on 2160 pixels 21.4 / 31.8; 169 -> 23 on 8712 30.5 / 25.2; 7 x 7, 193 -> 15 on 11236, K = 9457, 35.4 / 40.5).
inline bool kgroup_ragged_rule(const KGroupCall& c) {
  const int64_t t = tiles_of(c.M, c.N, 32, 32), kbytes = (int64_t)c.K * c.eb, row = (int64_t)c.N * c.eb;
  if (c.conv) {
    if (kbytes < (row > 32 ? 200 : c.Cin % 16 == 0 ? 800 : c.Cin % 4 == 0 ? 320 : 200)) return false;
    if (t <= 256) return c.splits <= 1 || kbytes <= 3500;
    return t <= 448 && kbytes >= (c.Cin % 16 == 0 ? 2400 : 1200) && (c.splits <= 1 || kbytes <= (row <= 32 ? 4500 : 2400));
  }
  if (kbytes < 16) return false;
  if (t <= 256) return c.splits <= 1 || (kbytes <= 3500 && (row <= 64 || kbytes <= 2432 + 6 * t));
  if (t > 448 || (c.splits > 1 && kbytes > 2048)) return false;
  if (c.eb == 2) return kbytes <= 8192;
  if (c.b_along_k) return c.a_along_k || kbytes <= 3500;
  return kbytes <= (c.a_along_k ? 2200 : 1408);
}

// Whether an uncut product on operands aligned to 4 bytes (dword_operands) that the shared tiles leave takes the direct-to-LDS
// tiles; otherwise the any-alignment kernels, in us (there / here).  Between one and two rounds of 64 x 64 tiles those have a
// tile of 128 x 64, one to a compute unit (828 x 2276 x 4028 21.1 / 26.4, int32 904 x 1380 x 2668 13.4 / 16.6, bf16 1184 x
// 1364 x 1610 15.7 / 18.4, A^T 816 x 1516 x 2808 14.8 / 18.3, B^T 1600 x 980 x 940 6.7 / 7.8).  Up to three tiles to a compute
// unit, the last K tile of these costs more than its products (2639 x 212 x 64 3.9 / 4.2, bf16 2107 x 1120 x 36 5.8 / 6.5; 1146 x
// 2564 x 2076 15.8 / 14.7), and longer, up to four, where both operands end inside a chunk (B^T 535 x 1672 x 28 3.9 / 4.4,
// 1564 x 536 x 772 5.5 / 6.0, 7077 x 460 x 156 6.1 / 6.7, 3513 x 788 x 1032 level).
inline bool dword_tiles_rule(int32_t M, int32_t N, int64_t kbytes, bool both_along_k) {
  const int64_t t64 = tiles_of(M, N, 64, 64);
  if (t64 > PLAN_CUS && tiles_of(M, N, 128, 64) <= PLAN_CUS) return false;
  return both_along_k ? t64 > 4 * PLAN_CUS || kbytes >= 1024 : t64 > 3 * PLAN_CUS || kbytes >= 192;
}

// Whether a product of 256 x 256 tiles, uncut, runs on the interleaved K loop (one wave to a SIMD, 16 x 16 MFMA tiles) instead of the
// ping-pong one.  Its gain is that of the power limit, which compute units without a tile lift; one wave to a SIMD works through fill
// and output stage alone (and, behind a prefetch, moves accumulators and in the plain int8 form waits for spilled registers).  So K
// has to be the longer, the more units idle in the last round, and the fewer rounds there are.  Ping-pong / here, times as fast, means over some 8000 random
// products of 130 to 800 tiles, by tiles a round (168, 192, 212 and from 232 on):
//   bytes of K      900 to 1300          1800 to 2560          3500 to 6000
//   int8            .90 .93 .94 .94      .95  .98 1.00 1.03    1.01 1.02 1.06 1.09
//     several       .96 .92 .91 .93     1.02  .99  .99 1.02    1.08 1.05 1.05 1.08   (2560 to 3500: 1.05 1.02 1.02 1.03)
//   B^T             .99 .99 1.00 1.01   1.00 1.00 1.01 1.00    1.01 1.01 1.02 1.06
//     several      1.00 .99 1.00 1.01   1.01 1.01 1.01 1.02    1.03 1.02 1.02 1.03
//   int32               .94 .95 .99           .98 1.00 1.04         1.03 1.07 1.09
//     several       .96 .98 .98 1.00    1.00 1.02 1.02 1.07    1.06 1.08 1.08 1.09
//   bf16            .88 .91 .94 .95      .92  .94  .97 .99      .97  .97 1.03 1.03   (on dwords .01 to .03 more)
//     several           .93 .94 .95      .98  .97  .99 1.02    1.01 1.06 1.10 1.08
//   A^T B^T        1.01 1.01 1.03 1.02  1.04 1.08 1.04 1.05    1.04 1.04 1.07 1.07
//     several      1.02 1.03 1.05 1.01  1.06 1.04 1.05 1.06    1.05 1.02 1.03 1.03
// Past the lines below 1.05 in the mean of 2942, 15 of them slower by 2.5 to 4.3 %.  8192^3 int8 441 / 380 us, 8192 x 8192 x 1024 bf16
// 132.5 / 115.5.  A^T alone gains nothing (4096 x 8192 x 4096 111.6 / 109.6, x 8192 210.7 / 212.2): neither operand's lines are
// requested twice there.  Lines of K and whole tiles alone held bf16 back by up to 9 % (3674 x 6792 x 616, 405 tiles, 46.7 / 51.5) and
// int8 by up to 6 % (5203 x 5376 x 2272 63.2 / 67.6).
inline bool interleaved_rule(int32_t M, int32_t N, int64_t kbytes, int eb, int out_bytes, bool trans_a, bool trans_b) {
  if (trans_a && !trans_b) return false;
  const int64_t tiles = tiles_of(M, N, 256, 256), rounds = (tiles + PLAN_CUS - 1) / PLAN_CUS;
  if (tiles < 184) return false;
  const bool one = rounds == 1, plain_i8 = eb == 1 && out_bytes == 1 && !trans_b;
  // bytes of K on full rounds, and how many more for a unit that idles in the last one: its share of the launch, and of the lifted
  // limit, falls with the rounds
  const int64_t least = eb == 2 || out_bytes == 4 ? (one ? 2560 : 1536) : plain_i8 ? (one ? 1280 : 2560) : trans_a ? (one ? 1024 : 512) : 1024;
  const int64_t per_idle = eb == 2 ? 96 : out_bytes == 4 ? (one ? 24 : 48) : plain_i8 ? (one ? 48 : 0) : trans_a ? (one ? 8 : 0) : 32;
  return (kbytes - least) * rounds * rounds >= per_idle * (rounds * PLAN_CUS - tiles);
}

// The same question for an int8 product on 128 x 256 tiles (four waves of 64 x 128 instead of eight of 64 x 64, a second wave to a
// SIMD under whose products the output stage of the first hides).  86 random products, us before / interleaved: on one tile a
// compute unit 2688 x 1600 x 512 7.5 / 8.6, 3648 x 1344 x 1024 10.7 / 11.3, K = 1536 and 1792 0.97 to 1.08 times as fast, from 2048
// on 0.99 to 1.16 (3616 x 1856 x 4096 32.4 / 30.1); on more 5088 x 3520 x 512 21.1 / 21.7, x 1024 level, from 1280 on 1.03 to 1.16
// (4304 x 5504 x 1536 43.3 / 40.9).  With a hundred idle units one round needs K of some 2600 (1334 x 3456 x 2512, 154 tiles, 0.95
// times as fast; 55 others from 2048 on 1.04 in the mean).  bf16 on 256 x 128 tiles the same way 0.88 to 1.09, up and down at any K: not
// taken.
inline bool interleaved_128x256_rule(int32_t M, int32_t N, int32_t K) {
  const int64_t tiles = tiles_of(M, N, 128, 256);
  return tiles > PLAN_CUS ? K >= 1280 : K >= 2048 && K >= 1792 + 8 * (PLAN_CUS - tiles);
}

// A^T B^T products on one round of those tiles, where the 128 x 128 ones that they had make two, and that cover little more than
// the output.  46 random ones 1.02 to 1.28 times as fast (us before / here: 2640 x 2224 x 576 11.8 / 9.9, 848 x 5984 x 768 13.1 / 11.2, 2720
// x 1728 x 1024 16.0 / 12.5, 736 x 5424 x 2304 24.2 / 19.7, 6448 x 1184 x 5120 52.3 / 42.1); 130 tiles where 250 of 128 x 128 fill the chip
// 1216 x 3136 x 5120 27.2 / 38.1; a third of the tiles' area outside 6240 x 576 x 768 7.0 / 9.9; on more than a round level.  B^T alone
// is up and down (2560 x 2832 x 576 11.4 / 10.1, 1920 x 3200 x 2048 18.2 / 19.5, 3008 x 5824 x 1536 39.8 / 43.4): not taken.
inline bool interleaved_at_bt_rule(int32_t M, int32_t N, int32_t K) {
  const int64_t tiles = tiles_of(M, N, 128, 256);
  return tiles <= PLAN_CUS && tiles_of(M, N, 128, 128) > PLAN_CUS && K >= 512 && tiles * (128 * 256) * 4 <= (int64_t)M * N * 5;
}

}  // namespace ac
