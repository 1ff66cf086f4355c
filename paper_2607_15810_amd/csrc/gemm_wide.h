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
  double time;
};

// The estimated time in the panel schedule's unit (panel_sched.h): rounds of the
// 256 CUs, a tile of up to 128 rows 6.8, a taller one, whatever its height, 10.5.
// A round lasts as long as its tallest tile, so each CU is taken to meet
// one tall tile if there is any (64 experts of 110 +- 10 rows, three tiles wide: one
// round, and 104 us against 87 with the panel kernel for the few above 128).
inline double wide_time(int64_t rows, int E, int ntn, double nst) {
  const double mean = (double)rows / E, sd = std::max(0.5, sqrt(mean));
  const double n = std::max(qdp::pn_tiles(mean, sd, E, 256.0, 0.0), 1.0 / E);
  const double tall = qdp::pn_tiles(mean, sd, E, 256.0, 128.0);
  const double any = E == 1 ? (tall > 0.0 ? 1.0 : 0.0) : 1.0 - std::exp(-tall * E);
  const double r = qdp::pn_rounds(n * E, ntn);
  return (6.8 + 4.0 / nst) * r + 3.7 * std::min(r, r * tall / n + any);
}

// The weights must carry fragment-ordered scales.
WdPlan wide_plan(int64_t rows, int64_t a_rows, int E, int64_t N, int64_t K);
void launch_wide(const GemmArgs &p, int epilogue, const WdPlan &pl, hipStream_t s);

}  // namespace qdw
