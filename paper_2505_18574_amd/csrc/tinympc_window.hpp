// LDS window of a wave of tinympc_forward_quad_kernel (tinympc_f32.hip): sixteen problems, d / u and behind it the
// trajectory.  Plain host arithmetic, which the kernel shares and a test can compile by itself.
#pragma once
#include <stdint.h>

namespace ac {

constexpr int TMPC_QUAD_WINDOW = 4096;  // floats of a wave's window at most: ten waves to a compute unit
constexpr int TMPC_QUAD_MATRICES = 256;  // ... at least: a matrix passes through it on its way into registers

// Where things lie in the window, in floats.  WHOLE holds the d / u and the states x[0 .. horizon] of the whole horizon;
// otherwise it holds `chunk` steps of d / u and the states after them (x[0] has no place in a chunk).
struct TmpcLayout {
  int dpitch, xpitch;  // from one problem to the next
  int xwin;            // start of the trajectory
};
constexpr TmpcLayout tmpc_layout(int nx, int nu, int horizon, int chunk, bool whole) {
  return {chunk * nu, (whole ? horizon + 1 : chunk) * nx, 16 * chunk * nu};
}

// From one problem to the next in memory: `steps` of `size` values each, more than 2^31 of them at long horizons.
constexpr int64_t tmpc_pitch(int64_t steps, int size) { return steps * size; }

struct TmpcWindow {
  bool whole;
  int chunk;   // steps that go through the window at a time (whole: the horizon)
  int floats;  // of the window
};
// Whole as long as all of it fits.  A chunk may be as long as the horizon: the states x[0], which only the whole form
// keeps in the window, can be what does not fit.
constexpr TmpcWindow tmpc_window(int nx, int nu, int horizon, bool trajectory) {
  const int per_step = 16 * (nu + (trajectory ? nx : 0));
  const int64_t all = (int64_t)horizon * per_step + (trajectory ? 16 * nx : 0);
  const bool whole = all + 3 <= TMPC_QUAD_WINDOW;
  const int chunk = whole ? horizon : (TMPC_QUAD_WINDOW - 3) / per_step;
  const int used = whole ? (int)all : chunk * per_step;
  return {whole, chunk, used < TMPC_QUAD_MATRICES ? TMPC_QUAD_MATRICES : used};
}

}  // namespace ac
