// Shape of the stencil's blocked-step form (k_jacobi_tile and
// k_jacobi_one_window in stencil.hip): which windows, how many launches, how
// many steps each.  Plain host arithmetic with no HIP in it, so that a test
// without a GPU can evaluate it.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace redsum {

constexpr int kTileLanes = 64;  // lanes of a wavefront
constexpr int kTileWG = 256;    // four wavefronts, one per SIMD; they do not cooperate

// Values per lane of the window kernels.
constexpr int kTileValues[] = {2, 4, 6, 8, 12, 16, 20, 24, 28, 36};

// One wavefront for the whole array: up to 64 x 8 interior values.
struct OneWindow {
  int v;
  double us_per_step;  // measured
};
constexpr OneWindow kOneWindows[] = {{2, 0.044}, {4, 0.064}, {8, 0.104}};

struct TilePlan {
  int v = 0;         // values per lane
  int launches = 0;  // 0: one launch per step instead; 1: the one-window kernel; else even, u and scratch alternating
  int k = 0;         // window margin: at least the steps of one launch
  int m = 0;         // interior values that a window advances
  int64_t waves = 0;
};

// Cost of a launch besides its steps: the kernel boundary, the ramp and the
// first load (2.2 us from 1 K to 64 K values), and the array's read and
// write.  While every wavefront is resident at once all of them load before
// they compute (about 10 TB/s beyond the 2.2 us, from the caches); beyond
// that the loads run under other wavefronts' steps at a large copy's rate,
// 4.8 TB/s (24 M values, 4 steps: 40 us), less for runs longer than 64 bytes
// per lane, whose loads and stores touch more lines at a time.
constexpr double kTileLaunchUs = 2.2;
constexpr double kTileCachedBytesPerUs = 10e6;
constexpr double kTileStreamBytesPerUs = 4.8e6;

// Cycles per VALU operation and SIMD with w wavefronts resident on it
// (measured: 4 M and 1 M values with windows of 12 to 36 values per lane).
inline double tile_cycles_per_op(double w) { return w <= 1 ? 4.6 : w <= 2 ? 3.2 : w <= 3 ? 2.9 : 2.75; }

// One or two steps on this many values and more run as one launch per step:
// two passes over the array either way, and whole-array streams pass at 6.5
// TB/s where windows pass at 4.8 (one step, us as launches per step / as
// windows: 1 M values 6.4 / 6.1, 2 M 7.5 / 8.5, 4 M 11.9 / 16.7, 16 M 40 /
// 68, 24 M 58 / 79, 100 M 320 / 355; two steps 6.4 / 6.1, 8.4 / 8.6, 12.6 /
// 16.7, 42 / 67, 60 / 79, 334 / 353).  Three steps are four passes against
// two (4 M 24.4 / 16.6, 24 M 119 / 80).
constexpr int kStepLaunchMaxSteps = 2;
constexpr int64_t kStepLaunchMinValues = 2 << 20;

// The shape of the lowest modelled time for N interior values and `steps`
// steps.  More steps per launch save launches and widen the recomputed
// margins; a larger window has relatively narrower margins, but a small
// array then leaves SIMDs idle, and a step takes as long as the fullest SIMD
// (4 V operations per wavefront on it).
inline TilePlan plan_tiles(int64_t N, int steps, int cus, int64_t clock_khz) {
  TilePlan best;
  if (steps <= kStepLaunchMaxSteps && N >= kStepLaunchMinValues) return best;
  double best_us = 1e300;
  if (N <= 8 * kTileLanes)
    for (const OneWindow& k : kOneWindows)
      if (N <= (int64_t)k.v * kTileLanes) {
        best.v = k.v;
        best.launches = 1;
        best_us = kTileLaunchUs + k.us_per_step * steps;
        break;
      }
  const double cyc_us = clock_khz * 1e-3;
  for (const int v : kTileValues) {
    const int w_vals = kTileLanes * v;
    if (N < w_vals) break;
    // From the fewest launches whose margins leave a quarter of the window,
    // up in steps of about a third, eight candidates.  In 64 bits: steps may
    // be as large as an int holds.
    int64_t L = std::max<int64_t>(2, ((int64_t)steps + 24 * v - 1) / (24 * v));
    for (int c = 0; c < 8; ++c) {
      L += L & 1;
      const int per = (int)((steps + L - 1) / L);
      const int k = (per + 3) & ~3;  // keeps the block edges of interior windows on whole vectors
      const int m = w_vals - 2 * k;
      const int64_t waves = (N + m - 1) / m;
      const int64_t wgs = (waves + kTileWG / kTileLanes - 1) / (kTileWG / kTileLanes);
      const bool resident = wgs <= 8 * (int64_t)cus;
      const double load = resident ? (double)((wgs + cus - 1) / cus) : (double)wgs / cus + 0.5;
      const double step_us = per * load * (4 * v + 2) * tile_cycles_per_op(load) / cyc_us;
      double us;
      if (resident) {
        us = step_us + 8.0 * (double)N / kTileCachedBytesPerUs;
      } else {
        const double mem_us = 8.0 * (double)N / kTileStreamBytesPerUs * (v <= 16 ? 1.0 : v <= 20 ? 1.15 : 1.35);
        us = std::max(step_us, mem_us) + 0.2 * std::min(step_us, mem_us);
      }
      us = (double)L * (us + kTileLaunchUs);
      if (us < best_us) {
        best_us = us;
        best = TilePlan{v, (int)L, k, m, waves};
      }
      if (per <= 8) break;
      L += std::max<int64_t>(2, L / 3);
    }
  }
  return best;
}

}  // namespace redsum
