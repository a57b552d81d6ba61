// Forward pass of the TinyMPC primal update, batched over independent problems:
//   u[i]   = -Kinf . x[i] - d[i]
//   x[i+1] =  Adyn . x[i] + Bdyn . u[i]        i = 0 .. horizon-1
// Per problem the operation moves nx + horizon * nu floats in and horizon * nu out (plus the optional state
// trajectory): with the paper's sizes (12, 4, 5) that is 208 bytes (496 with the trajectory) for 2400 flop, so HBM
// bounds it.  Two families: the paper's sizes, at horizons up to its 5, run on the matrix units, sixteen problems to a
// 16 x 16 product (tinympc_forward_mfma_kernel); any other size or horizon, and unaligned arrays, on the vector ALU with
// four lanes per problem (tinympc_forward_quad_kernel).
#include "common.hpp"
#include "tinympc_window.hpp"

#include <type_traits>

namespace ac {

// The paper's state and control sizes (12, 4) on the matrix units.  With u[i] substituted into the state update a
// step is one 16 x 16 product on the stacked vector z = [x[i] (12); d[i] (4)] of each problem:
//   [x[i + 1]; u[i]] = M . z,     M = [Adyn - Bdyn Kinf, -Bdyn; -Kinf, -I]
// v_mfma_f32_16x16x4_f32 takes a 16 x 4 and a 4 x 16 operand, one value per lane: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16], and returns D[4 (l / 16) + v][l % 16] in register v = 0..3.  Sixteen problems are the columns.
// The sum over the 16 rows of z is order-free, so instruction c of a product takes rows 4 g + c (g = l / 16): the
// four registers a lane RECEIVES from one product (rows 4 g + 0..3 of its problem) are exactly the four values it
// FEEDS to the next, with no data movement in between; only the matrix operands are laid out to match (lane
// (m, g) holds column 4 g + c of row m for instruction c: four registers per matrix for the whole kernel).
// A wave owns NB such column blocks of consecutive problems; lanes g < 3 carry x, lanes g == 3 carry d and u.
// Some 500 instructions per 64 problems, 80 of them MFMAs, against 2100 on the vector ALU with one problem per
// lane.  Sums are fp32 throughout, in the matrix unit's order and with the closed-loop matrix formed first: equal to
// the recurrence in exact arithmetic, a few ulp from the ascending chains of the other kernels in fp32.
//
// Memory: the inputs and outputs of a wave's 64 problems are four contiguous runs (x0 3 KB, d and u 5 KB each, the
// trajectory 18 KB), but a lane's share of them is 16 bytes per step: stored as produced, a memory line is completed
// by instructions a whole step apart and leaves the L2 half written in between (58 us for 262144 problems; 39 us
// with the results held in registers and stored back to back at the end).  d is therefore loaded, and u and the
// trajectory are stored, as whole runs of 16 bytes per lane through a wave-private LDS window (u overwrites d in place,
// step by step; the trajectory goes block by block through a second window).  The results of a block stay in registers
// until then, which fixes the horizon H at compile time: the paper's 5 and the shorter ones.
constexpr int TMPC_H = 5;

// NB: column blocks (of sixteen problems) per wave; WAVES per workgroup.  Four blocks hide a block's chain of 20 MFMAs behind
// three others and are right once every compute unit has work; a small batch is one such chain after three memory
// latencies, and one block to a wave, one wave to a workgroup, shortens the chain and spreads it over the chip (100
// problems 7.0 -> 4.1 us, 4000 7.6 -> 4.4, up to four such waves per compute unit: 16384 problems, 5.0 us).
template <bool WITH_X, int H, int NB, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) tinympc_forward_mfma_kernel(const TinyMpcParams p) {
  constexpr int NX = 12, NU = 4, PB = 16 * NB;            // PB: problems of a wave-block
  constexpr int DN = (PB * H + 63) / 64;                  // 16-byte pieces of d per lane
  constexpr int XPITCH = 16 * (((H + 1) * NX / 4) | 1);   // LDS bytes per problem of a trajectory block, an odd number of pieces
  constexpr int WAVE_LDS = DN * 1024 + 16 * XPITCH;       // d / u window of PB problems + trajectory window of 16
  __shared__ __attribute__((aligned(16))) unsigned char tmpc_lds[WAVES * WAVE_LDS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, g = lane >> 4;
  // Wave-block k is problems PB k .. PB k + PB - 1; a wave takes blocks first, first + stride, ... (persistent
  // waves that request their next block's inputs before they compute and store the current one, so that loads,
  // products and stores of different blocks overlap; with one block per wave the whole chip loads, then
  // multiplies, then stores: 38 us for 262144 problems).
  const int64_t nblk = (p.batch + PB - 1) / PB, stride = (int64_t)gridDim.x * WAVES;
  int64_t blk = (int64_t)blockIdx.x * WAVES + wave;
  if (blk >= nblk) return;  // whole waves leave; no wave waits for another
  unsigned char* dwin = tmpc_lds + wave * WAVE_LDS;  // [PB problems][H][4] floats: d, then u
  unsigned char* xwin = dwin + DN * 1024;            // [16 problems][XPITCH]

  // inputs of a block: d as one contiguous run, 16 bytes per lane and instruction, and per column block the
  // lane's 16 bytes of x0 (lanes past the end re-read the last problem and store nothing).  Every byte is read once
  // and every result written once, so loads and stores carry the non-temporal hint (262144 problems: 27.0 -> 26.3 us
  // with the trajectory, 18.7 -> 16.0 us without)
  v4f din[DN], xin[NB];
  auto request = [&](int64_t k) {
    const int left = p.batch - k * PB < PB ? (int)(p.batch - k * PB) : PB;
    const v4f* src = (const v4f*)(p.d + k * PB * H * NU);
#pragma unroll
    for (int j = 0; j < DN; j++) {
      const int q = j * 64 + lane;
      din[j] = q < left * H ? __builtin_nontemporal_load(src + q) : (v4f){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int b = 0; b < NB; b++) {
      const int64_t q = k * PB + 16 * b + n;
      xin[b] = g < 3 ? __builtin_nontemporal_load((const v4f*)(p.x0 + (q < p.batch ? q : p.batch - 1) * NX + 4 * g)) : (v4f){0.f, 0.f, 0.f, 0.f};
    }
  };
  request(blk);

  // matrix operand of instruction c: row m = n, column k = 4 g + c of
  //   M = [ Adyn - Bdyn Kinf   -Bdyn ]     so that   M . [x[i]; d[i]] = [x[i + 1]; u[i]]
  //       [      -Kinf           -I  ]
  // (x[i + 1] = Adyn x[i] + Bdyn u[i] with u[i] = -Kinf x[i] - d[i] substituted; Adyn - Bdyn Kinf is formed here in
  // fp32, four fused multiply-adds per entry in ascending order).  Every lane loads from clamped positions and picks
  // afterwards: loads behind branches would wait for one another.
  float mat[4];
  {
    const int row = n < NX ? n : NX - 1, urow = n < NX ? 0 : n - NX;
    float bd[NU], ad[4], kf[NU][4];
#pragma unroll
    for (int j = 0; j < NU; j++) bd[j] = p.Bdyn[row * NU + j];
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const int k = g < 3 ? 4 * g + c : c;
      ad[c] = p.Adyn[row * NX + k];
#pragma unroll
      for (int j = 0; j < NU; j++) kf[j][c] = p.Kinf[j * NX + k];
    }
#pragma unroll
    for (int c = 0; c < 4; c++) {
      float closed = ad[c];
#pragma unroll
      for (int j = 0; j < NU; j++) closed = __builtin_fmaf(-bd[j], kf[j][c], closed);
      const float gain = urow == 0 ? kf[0][c] : urow == 1 ? kf[1][c] : urow == 2 ? kf[2][c] : kf[3][c];
      mat[c] = n < NX ? (g < 3 ? closed : -bd[c]) : (g < 3 ? -gain : (c == urow ? -1.f : 0.f));
    }
  }

  for (; blk < nblk; blk += stride) {
    const int nvalid = p.batch - blk * PB < PB ? (int)(p.batch - blk * PB) : PB;
#pragma unroll
    for (int j = 0; j < DN; j++) *(v4f*)(dwin + 16 * (j * 64 + lane)) = din[j];
    v4f z[NB];  // lanes g < 3: x0 rows 4 g .. 4 g + 3; lanes g == 3 take d[0] below
#pragma unroll
    for (int b = 0; b < NB; b++) z[b] = xin[b];
    if (blk + stride < nblk) request(blk + stride);
    v4f hist[H + 1][NB];  // lanes g < 3: the lane's rows of x[0 .. H]
#pragma unroll
    for (int b = 0; b < NB; b++) hist[0][b] = z[b];

    // z = [x[i]; d[i]]: lanes g == 3 take d[i] from the window
    auto d_of = [&](int b, int i) { return *(const v4f*)(dwin + (16 * b + n) * (H * 16) + i * 16); };
#pragma unroll
    for (int b = 0; b < NB; b++)
      if (g == 3) z[b] = d_of(b, 0);
#pragma unroll
    for (int i = 0; i < H; i++) {
      v4f acc[NB];
#pragma unroll
      for (int b = 0; b < NB; b++) acc[b] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < 4; c++)  // the column blocks are independent: their instructions alternate
#pragma unroll
        for (int b = 0; b < NB; b++) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(mat[c], z[b][c], acc[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < NB; b++) {
        if (g == 3) {  // rows 12..15: u[i], into the place of d[i]; then d[i + 1]
          *(v4f*)(dwin + (16 * b + n) * (H * 16) + i * 16) = acc[b];
          if (i + 1 < H) z[b] = d_of(b, i + 1);
        } else {       // rows 0..11: x[i + 1]
          z[b] = acc[b];
          hist[i + 1][b] = acc[b];
        }
      }
    }

    // u: the window, in memory order, 16 bytes per lane (LDS serves a wave's operations in order: the reads below
    // see the writes above without a wait of their own beyond the compiler's)
    {
      v4f* dst = (v4f*)(p.u + blk * PB * H * NU);
      const int pieces = nvalid * H;
#pragma unroll
      for (int k = 0; k < DN; k++) {
        const int q = k * 64 + lane;
        if (q < pieces) __builtin_nontemporal_store(*(const v4f*)(dwin + 16 * q), dst + q);
      }
    }
    if constexpr (WITH_X) {
      constexpr int XROW = (H + 1) * NX * 4;  // bytes of trajectory per problem
      constexpr int PPB = XROW / 16;          // 16-byte pieces per problem
#pragma unroll
      for (int b = 0; b < NB; b++) {
        if (g < 3) {
#pragma unroll
          for (int i = 0; i <= H; i++) *(v4f*)(xwin + n * XPITCH + i * (NX * 4) + g * 16) = hist[i][b];
        }
        v4f* dst = (v4f*)(p.x_out + (blk * PB + 16 * b) * (int64_t)(H + 1) * NX);
        const int left = nvalid - 16 * b;  // problems of this block that exist
        const int pieces = (left < 0 ? 0 : left > 16 ? 16 : left) * PPB;
#pragma unroll
        for (int k = 0; k < (16 * PPB + 63) / 64; k++) {
          const int q = k * 64 + lane;  // piece q of the block: problem q / PPB, piece q % PPB of its rows
          if (q < pieces) __builtin_nontemporal_store(*(const v4f*)(xwin + (q / PPB) * XPITCH + (q % PPB) * 16), dst + q);
        }
      }
    }
  }
}

// Any 1 <= nx, nu <= 16 and any alignment: the recurrence as written, on the vector ALU, four lanes (a quad) to a
// problem and sixteen problems to a wave.  Lane q of a quad owns the state rows q + 4 i and the control rows q + 4 j and
// keeps its rows of the three matrices in registers for the whole kernel (RX = ceil(nx / 4), RU = ceil(nu / 4): at most
// 192 values); x[c] reaches the quad by a DPP quad broadcast, which all of the lane's row sums share.  Every sum is still
// one fused multiply-add chain in ascending index order from zero; indices beyond nx / nu add 0 * 0 (the rows there are set
// to zero after every step).
//
// One lane per problem, which this replaces, keeps the matrices in LDS: one LDS read per multiply-add, and a chain of
// nx (nx + 2 nu) of both per step that a small batch has nothing to hide behind.  With the trajectory, before -> now:
// 100 problems of (10, 2, 4) 27.5 -> 4.5 us, of (13, 8, 8) 115 -> 7.0, of (12, 4, 8) 12.0 -> 5.6; 262144 of them 94 -> 28,
// 563 -> 70 and 101 -> 44 us (5 TB/s: 16, 54 and 39).  Here a step is 4 RX broadcasts and 4 RX (RX + RU) + 4 RU RX multiply-adds, RX + RU of
// them independent.
//
// d comes in and u and the trajectory leave as whole contiguous runs through a wave-private LDS window (u overwrites d
// in place; tinympc_window.hpp).  A horizon too long for the window goes through it `chunk` steps at a time, a run per
// problem.  WHOLE: all of it is in the window at once.
template <int RX, int RU, bool WHOLE>
__global__ void __launch_bounds__(256) tinympc_forward_quad_kernel(const TinyMpcParams p, const int window, const int chunk) {
  extern __shared__ __attribute__((aligned(16))) float tmpc_quad_lds[];
  const int nx = p.nx, nu = p.nu, H = p.horizon;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int q = lane & 3, pr = lane >> 2;
  const int64_t nblk = (p.batch + 15) / 16, stride = (int64_t)gridDim.x * waves;
  const bool traj = p.x_out != nullptr;
  const TmpcLayout at = tmpc_layout(nx, nu, H, chunk, WHOLE);
  const int dpitch = at.dpitch, xpitch = at.xpitch;
  float* dwin = tmpc_quad_lds + wave * window;  // [16 problems][chunk][nu]: d, then u (before that: the matrices)
  float* xwin = dwin + at.xwin;
  const int64_t drun = tmpc_pitch(H, nu), xrun = tmpc_pitch((int64_t)H + 1, nx);
  float *dmine = dwin + pr * dpitch, *xmine = xwin + pr * xpitch;

  // The matrices pass through the wave's LDS window, padded with zeros to whole fours, so that a lane picks its rows up
  // 16 bytes at a time (entry by entry from memory it is 192 loads and their addresses: 16 us of a 21 us launch).
  float a[RX][4 * RX], k[RU][4 * RX], b[RX][4 * RU];
  auto rows_of = [&](const float* m, int rows, int cols, auto& reg, auto rc, auto cc) {
    constexpr int R = decltype(rc)::value, C = decltype(cc)::value, PC = C == 3 ? 4 : C;  // padded size / 4 (columns: a power of two)
    float v[(16 * R * PC + 63) / 64];
#pragma unroll
    for (int e = 0; e < (16 * R * PC + 63) / 64; e++) {
      const int i = e * 64 + lane, r = i / (4 * PC), c = i % (4 * PC);
      const float x = m[(r < rows ? r : rows - 1) * cols + (c < cols ? c : cols - 1)];
      v[e] = r < rows && c < cols ? x : 0.f;
    }
#pragma unroll
    for (int e = 0; e < (16 * R * PC + 63) / 64; e++) dwin[e * 64 + lane] = v[e];
#pragma unroll
    for (int i = 0; i < R; i++)
#pragma unroll
      for (int c = 0; c < C; c++) {
        const v4f w = *(const v4f*)(dwin + (q + 4 * i) * (4 * PC) + 4 * c);
#pragma unroll
        for (int e = 0; e < 4; e++) reg[i][4 * c + e] = w[e];
      }
  };
  constexpr std::integral_constant<int, RX> rx{};
  constexpr std::integral_constant<int, RU> ru{};
  rows_of(p.Adyn, nx, nx, a, rx, rx);
  rows_of(p.Kinf, nu, nx, k, ru, rx);
  rows_of(p.Bdyn, nx, nu, b, rx, ru);

  auto copy = [&](float* dst, const float* src, int count) {  // one contiguous run, 16 bytes per lane where both ends allow it
    const bool wide = ((((uintptr_t)dst) | ((uintptr_t)src)) & 15) == 0;
    const int fours = wide ? count & ~3 : 0;
#pragma unroll 4
    for (int i = lane * 4; i < fours; i += 256) *(v4f*)(dst + i) = *(const v4f*)(src + i);
#pragma unroll 4
    for (int i = fours + lane; i < count; i += 64) dst[i] = src[i];
  };
  // One run of `count` values per problem.  Value i of all of them is number i - r count of run r = i / count, by one
  // multiply: 16 runs fit the window, so count <= 255 and i * (count * magic - 2^20) < 2^20.
  auto copy_runs = [&](float* dst, int64_t dst_pitch, const float* src, int64_t src_pitch, int runs, int count) {
    const unsigned magic = (1u << 20) / (unsigned)count + 1u;
#pragma unroll 8
    for (int i = lane; i < runs * count; i += 64) {
      const int r = (int)(((unsigned)i * magic) >> 20), e = i - r * count;
      dst[r * dst_pitch + e] = src[r * src_pitch + e];
    }
  };

  for (int64_t blk = (int64_t)blockIdx.x * waves + wave; blk < nblk; blk += stride) {  // no wave waits for another
    const int64_t b0 = blk * 16;
    const int nvalid = p.batch - b0 < 16 ? (int)(p.batch - b0) : 16;
    const bool live = pr < nvalid;
    const int64_t prob = b0 + (live ? pr : 0);
    float x[RX], u[RU];
#pragma unroll
    for (int i = 0; i < RX; i++) x[i] = q + 4 * i < nx ? p.x0[prob * nx + q + 4 * i] : 0.f;
    if (traj) {
#pragma unroll
      for (int i = 0; i < RX; i++)
        if (live && q + 4 * i < nx) {
          if constexpr (WHOLE) xmine[q + 4 * i] = x[i];
          else p.x_out[prob * xrun + q + 4 * i] = x[i];
        }
    }
    for (int s0 = 0, steps = 0; s0 < H; s0 += steps) {
      steps = H - s0 < chunk ? H - s0 : chunk;
      if constexpr (WHOLE) copy(dwin, p.d + b0 * drun, nvalid * H * nu);
      else copy_runs(dwin, dpitch, p.d + b0 * drun + (int64_t)s0 * nu, drun, nvalid, steps * nu);
      float* xrow = xmine + (WHOLE ? nx : 0);
      for (int step = 0; step < steps; step++) {
        float dv[RU], su[RU], sx[RX];
#pragma unroll
        for (int j = 0; j < RU; j++) dv[j] = q + 4 * j < nu ? dmine[step * nu + q + 4 * j] : 0.f, su[j] = 0.f;
#pragma unroll
        for (int i = 0; i < RX; i++) sx[i] = 0.f;
#pragma unroll
        for (int c = 0; c < 4 * RX; c++) {
          const float v = quad_broadcast(x[c >> 2], c & 3);
#pragma unroll
          for (int j = 0; j < RU; j++) su[j] = __builtin_fmaf(k[j][c], v, su[j]);
#pragma unroll
          for (int i = 0; i < RX; i++) sx[i] = __builtin_fmaf(a[i][c], v, sx[i]);
        }
#pragma unroll
        for (int j = 0; j < RU; j++) {
          u[j] = q + 4 * j < nu ? -su[j] - dv[j] : 0.f;
          if (q + 4 * j < nu) dmine[step * nu + q + 4 * j] = u[j];
        }
        // the state after the last control is not needed for u; it is only produced when the trajectory is asked for
        if (s0 + step + 1 < H || traj) {
          float t[RX];
#pragma unroll
          for (int i = 0; i < RX; i++) t[i] = 0.f;
#pragma unroll
          for (int c = 0; c < 4 * RU; c++) {
            const float v = quad_broadcast(u[c >> 2], c & 3);
#pragma unroll
            for (int i = 0; i < RX; i++) t[i] = __builtin_fmaf(b[i][c], v, t[i]);
          }
#pragma unroll
          for (int i = 0; i < RX; i++) {
            x[i] = q + 4 * i < nx ? sx[i] + t[i] : 0.f;  // (rows beyond nx: 0 times an infinite state is no zero)
            if (traj && q + 4 * i < nx) xrow[step * nx + q + 4 * i] = x[i];
          }
        }
      }
      if constexpr (WHOLE) {
        copy(p.u + b0 * drun, dwin, nvalid * H * nu);
        if (traj) copy(p.x_out + b0 * xrun, xwin, nvalid * (H + 1) * nx);
      } else {
        copy_runs(p.u + b0 * drun + (int64_t)s0 * nu, drun, dwin, dpitch, nvalid, steps * nu);
        if (traj) copy_runs(p.x_out + b0 * xrun + (int64_t)(s0 + 1) * nx, xrun, xwin, xpitch, nvalid, steps * nx);
      }
    }
  }
}

template <int RX, int RU>
static hipError_t launch_quad(const TinyMpcParams& p, hipStream_t stream) {
  const TmpcWindow w = tmpc_window(p.nx, p.nu, p.horizon, p.x_out != nullptr);
  const int64_t blocks16 = (p.batch + 15) / 16;
  // one-wave workgroups until every compute unit has four: a small batch then spreads over the chip
  const int waves = blocks16 >= 4 * (int64_t)compute_units() ? 4 : 1;
  const int64_t most = (int64_t)compute_units() * 16 / waves;  // persistent beyond that: the matrices are loaded once per wave
  const int64_t wgs = (blocks16 + waves - 1) / waves;
  const dim3 grid((unsigned)(wgs < most ? wgs : most)), block(64 * waves);
  const size_t lds = (size_t)waves * w.floats * sizeof(float);
  if (w.whole) return launch_kernel(tinympc_forward_quad_kernel<RX, RU, true>, grid, block, lds, stream, p, w.floats, w.chunk);
  return launch_kernel(tinympc_forward_quad_kernel<RX, RU, false>, grid, block, lds, stream, p, w.floats, w.chunk);
}

template <int H, int NB, int WAVES>
static hipError_t launch_mfma_form(const TinyMpcParams& p, hipStream_t stream) {
  const int64_t blks = (p.batch + 16 * NB - 1) / (16 * NB), wgs = (blks + WAVES - 1) / WAVES;
  // one persistent workgroup of four waves per compute unit (27.3 us for 262144 problems; two, three, four: 31.1,
  // 33.0, 34.9 us)
  const int64_t slots = (int64_t)compute_units() * (4 / WAVES);
  const dim3 grid((unsigned)(wgs < slots ? wgs : slots)), block(64 * WAVES);
  if (p.x_out) return launch_kernel(tinympc_forward_mfma_kernel<true, H, NB, WAVES>, grid, block, 0, stream, p);
  return launch_kernel(tinympc_forward_mfma_kernel<false, H, NB, WAVES>, grid, block, 0, stream, p);
}

template <int H>
static hipError_t launch_mfma(const TinyMpcParams& p, hipStream_t stream) {
  return p.batch <= 16 * 4 * (int64_t)compute_units() ? launch_mfma_form<H, 1, 1>(p, stream) : launch_mfma_form<H, 4, 4>(p, stream);
}

hipError_t launch_tinympc_forward(const TinyMpcParams& p, hipStream_t stream) {
  if ((p.batch + 255) / 256 > 0x7fffffffLL) return hipErrorInvalidValue;
  const bool aligned16 = ((((uintptr_t)p.x0) | ((uintptr_t)p.d) | ((uintptr_t)p.u) | ((uintptr_t)p.x_out)) & 15) == 0;
  // The paper's sizes up to its horizon, where a call is bound by the bytes it moves; 262144 problems on the vector ALU and
  // here: horizon 1 12.3 and 6.7 us, 4 21.5 and 13.7, with the trajectory 19.7 and 11.2, 29.8 and 22.1.  (Beyond 5, where the
  // registers of a block's states run out, the vector ALU is ahead of matrix units that store state by state: horizon 6
  // without the trajectory 41 us so and 28.7, 40 322 and 126, with it in chunks 16 213 and 177, 40 596 and 398; 100 problems
  // of horizon 8 11.2 and 5.2, of 100 with the trajectory 115 and 66.)
  if (p.nx == 12 && p.nu == 4 && p.horizon <= TMPC_H && aligned16) {
    switch (p.horizon) {
      case 1: return launch_mfma<1>(p, stream);
      case 2: return launch_mfma<2>(p, stream);
      case 3: return launch_mfma<3>(p, stream);
      case 4: return launch_mfma<4>(p, stream);
      case TMPC_H: return launch_mfma<TMPC_H>(p, stream);
    }
  }
  switch (4 * ((p.nx - 1) / 4) + (p.nu - 1) / 4) {
#define AC_QUAD(RX, RU) \
  case 4 * (RX - 1) + RU - 1: return launch_quad<RX, RU>(p, stream);
    AC_QUAD(1, 1) AC_QUAD(1, 2) AC_QUAD(1, 3) AC_QUAD(1, 4)
    AC_QUAD(2, 1) AC_QUAD(2, 2) AC_QUAD(2, 3) AC_QUAD(2, 4)
    AC_QUAD(3, 1) AC_QUAD(3, 2) AC_QUAD(3, 3) AC_QUAD(3, 4)
    AC_QUAD(4, 1) AC_QUAD(4, 2) AC_QUAD(4, 3) AC_QUAD(4, 4)
#undef AC_QUAD
  }
  return hipErrorInvalidValue;
}

}  // namespace ac
