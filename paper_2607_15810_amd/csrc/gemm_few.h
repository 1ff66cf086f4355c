// Grouped W4A4 GEMM for a handful of rows (gemm_few_kernel): one request or a
// few decoding, eight experts each.  Launched from gemm.hip.
#pragma once
#include "gemm_args.h"

namespace qdf {

using qdg::GemmArgs;

constexpr int FW_WAVES = 4;              // waves per workgroup
constexpr int FW_N = 32;                 // weight rows per wave

struct FwPlan {
  bool ok;
  int split;    // log2 of the waves that share a block's K (1, 2 or 4)
  int nblk;     // blocks of FW_N weight rows (SwiGLU: half gate, half up) per expert
  int ngrp;     // workgroups per expert, FW_WAVES / split blocks each
  int grid;
};

FwPlan few_plan(int64_t rows, int E, int64_t N, int64_t K, int Ks, int epilogue, bool bitmap);
void launch_few(const GemmArgs &p, int epilogue, const FwPlan &pl, hipStream_t s);

}  // namespace qdf
