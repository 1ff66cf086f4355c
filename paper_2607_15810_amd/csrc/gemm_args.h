// Arguments and small device helpers shared by the grouped GEMM kernels.
#pragma once
#include "common.h"

namespace qdg {

using namespace qd;

struct GemmArgs {
  const uint8_t *a_codes;
  const uint8_t *a_scales;
  const float *a_gs;
  const int32_t *row_token;
  const int32_t *offsets;
  int E;
  int64_t rows;
  const uint8_t *w_codes;
  const uint8_t *w_scales;
  const uint8_t *w_sfrag;  // optional: the weight scales in fragment order
  const float *w_gs;
  int N;
  int K;
  const uint8_t *r_codes;
  const uint8_t *r_scales;
  const float *r_gs;
  const int32_t *sel;
  int Ks;
  const uint16_t *r_sel;   // f16 [a rows][ksa]: the residual at the selected channels
  int ksa;                 // row length of r_sel (Ks rounded up to 16)
  // bitmap mode (decode kernel only): r_bitmap [K / 32] marks S in place of
  // sel, and the kernel lists S into sel_out
  const uint32_t *r_bitmap;
  int32_t *sel_out;
  uint16_t *out;
  float *amax_part;
  int64_t amax_n;          // entries of amax_part (>= the grid; the rest are zeroed)
  // per-expert channel sets (panel and tile kernels): S of expert e at
  // sel + e * sel_stride, and r_sel indexed by grouped row instead of token
  int sel_stride;
  int rsel_rows;
};

// one maximum of |out| per workgroup into amax_part; workgroups also zero
// the entries past the grid, so every one of the amax_n entries is written
__device__ __forceinline__ void put_amax(const GemmArgs &p, float m) {
  if (p.amax_part && threadIdx.x == 0) {
    const int64_t g = (int64_t)gridDim.x * gridDim.y;
    const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    p.amax_part[b] = m;
    for (int64_t j = b + g; j < p.amax_n; j += g) p.amax_part[j] = 0.0f;
  }
}

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16 mfma32(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t word_of(uint4 v, int s) {
  return s == 0 ? v.x : (s == 1 ? v.y : (s == 2 ? v.z : v.w));
}

// silu(g) * u from f32 g and u: exp on the transcendental unit and one
// reciprocal (a few f32 ulp, far inside the bf16 rounding that follows)
__device__ __forceinline__ float swiglu_fast(float g, float u) {
  const float e = __builtin_amdgcn_exp2f(-g * 1.4426950408889634f);
  return g * __builtin_amdgcn_rcpf(1.0f + e) * u;
}

}  // namespace qdg
