// Grouped W4A4 GEMM without a residual on tiles of 256 x 256 (gemm_wide_kernel).
// Launched from gemm.hip.
#pragma once
#include "gemm_args.h"
#include "panel_sched.h"

namespace qdw {

using qdg::GemmArgs;

struct WdPlan {
  bool ok;
  int ntn, grid, lds;
};

// The estimated time in the panel schedule's unit (panel_sched.h): rounds of the
// 256 CUs, a tile of up to 128 rows 4.75, a taller one, whatever its height,
// 7.75.  A round lasts as long as its tallest tile, so each CU is taken to meet
// one tall tile if there is any (64 experts of 110 +- 10 rows, three tiles wide: one
// round, and 104 us against 87 with the panel kernel for the few above 128).
inline double wide_time(int64_t rows, int E, int ntn) {
  const double mean = (double)rows / E, sd = std::max(0.5, sqrt(mean));
  const double j0 = std::max(0.0, std::floor((mean - 8.0 * sd) / 256.0));
  double n = j0, tall = j0;
  for (double j = j0; 256.0 * j <= mean + 8.0 * sd; j += 1.0) {
    n += qdp::pn_above(256.0 * j, mean, sd, E);
    tall += qdp::pn_above(256.0 * j + 128.0, mean, sd, E);
  }
  n = std::max(n, 1.0 / E);
  const double any = E == 1 ? (tall > 0.0 ? 1.0 : 0.0) : 1.0 - std::exp(-tall * E);
  const double r = qdp::pn_rounds(n * E, ntn);
  return 4.75 * r + 3.0 * std::min(r, r * tall / n + any);
}

// panel_time: the panel kernel's estimate for the call.  The weights must carry
// fragment-ordered scales.
WdPlan wide_plan(int64_t rows, int64_t a_rows, int E, int64_t N, int64_t K, double panel_time);
void launch_wide(const GemmArgs &p, int epilogue, const WdPlan &pl, hipStream_t s);

}  // namespace qdw
