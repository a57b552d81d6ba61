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
// 192 8.0 -> 6.0, 8192 x 100000 x 80 466 -> 376; over 70 shapes of those ranges outside the fit 0.953 of the time (worst 1776 x
// 4560 x 5248 46.6 -> 48.5), over 80 of 8192 .. 900000 rows or columns 0.966 (worst 40811 x 128 x 864 13.7 -> 14.8).
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

}  // namespace ac
