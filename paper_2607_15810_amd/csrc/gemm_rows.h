// Grouped prefill GEMM over unpacked activations (gemm_rows_kernel): bf16
// activations times NVFP4 weights (the trainer-side W4A16 forward), or FP8
// activations times FP8 weights.
//
//  * Workgroup tile: up to 64 MF rows of one expert x 256 weight rows (SwiGLU:
//    128 gate rows and the matching 128 up rows), eight waves in a 2 x 4 grid,
//    each up to 32 MF rows x 64 weight rows of 32 x 32 fragments.  The tile
//    schedule is the NVFP4 panel kernel's (panel_sched.h): equal tiles to one
//    32-row fragment, experts of tall tiles first, one persistent workgroup per
//    CU, the stages of all its tiles one stream through an LDS ring.  (FP8 at 320
//    rows spills nine registers: the reload before the epilogue waits for the loads
//    in flight.)
//  * A stage is 128 bytes of each activation row (64 bf16 or 128 FP8 elements)
//    and the same elements of the weight rows, filled by direct global->LDS
//    loads of whole 128-byte lines.  The 16-byte pieces of a row are placed by a
//    row-dependent XOR, so the fragment reads are free of bank conflicts.  One
//    barrier per stage, where the last fragments it needs are in registers, so
//    that the next stage's first reads run under the last MFMAs.
//  * W4A16: MFMA k-step s takes the stage's elements 16 s .. 16 s + 15, half h
//    the 8 from 8 h on: the order of the general kernel (w4a16.hip), so that a
//    row's bits do not depend on which of the two runs.  A lane reads 16 bytes
//    of weight codes, elements 32 h .. 32 h + 31 of its row, and the two halves
//    swap words (two v_permlane32_swap per fragment and stage).  Each wave
//    decodes its weight fragments in registers: E2M1 x E4M3 has at most six
//    significant bits, so the f32 product is exact in bf16.
//    FP8: k-step s takes the stage's bytes 64 s .. 64 s + 63, half h 32 of them.
//
// What bounds it: for hundreds of rows per expert the wave's own chain of
// decode, fragment reads and MFMAs, two waves per SIMD (W4A16, 256 +- 16 rows on
// each of 128 experts, K = 2048, 1536 weight rows with SwiGLU: 345 -> 239 us =
// 0.86 PFLOP/s against 128 x 256 tiles that decoded through LDS between two
// barriers a stage; W2, K = 768, 2048 weight rows: 208 -> 137); for tens of rows
// HBM and the rounds of the chip (8 rows on each: 135 -> 86 us).  FP8, the same
// sizes, against 256 x 128 tiles of four waves and 64-byte pieces of rows: 211 ->
// 131 us = 1.57 PFLOP/s and 142 -> 102.  A cheaper SwiGLU at the same precision
// changed nothing beyond the noise (239 -> 235).
#pragma once
#include "gemm_args.h"
#include "panel_sched.h"

namespace qdr {

using namespace qd;
using namespace qdl;
using namespace qdp;
using qdg::f32x16;
using qdg::f32x2_t;
using qdg::bf16x2_t;
using qdg::word_of;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef int v8i __attribute__((ext_vector_type(8)));

struct RowsArgs {
  const uint8_t *a;          // [a_rows][K] bf16 or FP8
  const float *a_dec;        // FP8: scale per activation row
  const int32_t *row_token;
  const int32_t *offsets;
  int E;
  int64_t rows;
  const uint8_t *w_codes;    // [E][N][K / 2] E2M1 or [E][N][K] FP8
  const uint8_t *w_scales;   // W4A16: [E][N][K / 16]
  const float *w_dec;        // W4A16: {enc, dec} per expert; FP8: scale per weight row
  int N;
  int K;
  uint16_t *out;
};

template <bool FP8, int MF>
struct RwCfg {
  static constexpr int M = 64 * MF;
  static constexpr int BOFF = M * 128;                       // weight codes
  static constexpr int SOFF = BOFF + (FP8 ? 32768 : 8192);   // weight scales (W4A16)
  static constexpr int SLOT = SOFF + (FP8 ? 0 : 2048);
  static constexpr int NB = FP8 ? 4 : 1;                     // weight code loads per wave
  static constexpr int LPS = MF + NB + (FP8 ? 0 : 1);        // loads per wave and stage
};

struct RwLayout {
  int tok, dec, dummy, offs, mpre, perm, total;
};
// after the ring: the tokens and (FP8) the row and column scales of two tiles,
// the target of placeholder loads, the tile schedule
__host__ __device__ inline RwLayout rw_layout(bool fp8, int mf, int ns, int E) {
  RwLayout L{};
  int o = ns * (64 * mf * 128 + (fp8 ? 32768 : 10240));
  auto take = [&](int bytes) { const int at = o; o += (bytes + 15) & ~15; return at; };
  L.tok = take(2 * 64 * mf * 4);
  L.dec = take(fp8 ? 2 * (64 * mf + PN_N) * 4 : 0);
  L.dummy = take(256);
  L.offs = take((E + 1) * 4);
  L.mpre = take((E + 1) * 4);
  L.perm = take(E * 2);
  L.total = o;
  return L;
}

typedef const __attribute__((address_space(4))) RowsArgs *RwArgPtr;
__device__ __forceinline__ RwArgPtr rw_args() {
  RwArgPtr q = (RwArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(q));
  return q;
}

// 16-byte piece c of tile row r sits at piece c ^ rw_swz(r) of the row's 128
__device__ __forceinline__ int rw_swz(int r) { return (r >> 1) & 7; }

// weight row of the tile's row tb (0 past the last: never stored)
template <int EPI>
__device__ __forceinline__ int rw_wrow(int tb, int nt, int N) {
  if (EPI == QD_EPI_SWIGLU) {
    const int I = N >> 1, c = nt * 128 + (tb & 127);
    return c < I ? c + (tb < 128 ? 0 : I) : 0;
  }
  const int c = nt * PN_N + tb;
  return c < N ? c : 0;
}

__device__ __forceinline__ float rw_swiglu_w4a16(float g, float u) {
  return g / (1.0f + expf(-g)) * u;
}
__device__ __forceinline__ float rw_swiglu_fp8(float g, float u) {
  const float ex = __builtin_amdgcn_exp2f(-g * 1.4426950408889634f);
  return g * __builtin_amdgcn_rcpf(1.0f + ex) * u;
}

template <bool FP8, int MF, int EPI>
__global__ __launch_bounds__(PN_THREADS, 2) void gemm_rows_kernel(RowsArgs p, PnDeal deal,
                                                                  int ns) {
  using C = RwCfg<FP8, MF>;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ int sh_w[8];
  __shared__ int sh_c[8][2 * MF + 1];
  const int tid = threadIdx.x, lane = tid & 63, w = (int)uni((uint32_t)tid >> 6);
  const int N = p.N, E = p.E;
  const int kab = FP8 ? p.K : 2 * p.K;          // bytes of an activation row
  const int kwb = FP8 ? p.K : p.K >> 1;         // of a weight row
  const int nst = kab >> 7;
  const RwLayout L = rw_layout(FP8, MF, ns, E);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  int32_t *offs = reinterpret_cast<int32_t *>(lds + L.offs);
  int32_t *mpre = reinterpret_cast<int32_t *>(lds + L.mpre);
  uint16_t *perm = reinterpret_cast<uint16_t *>(lds + L.perm);
  const int32_t *tokb = reinterpret_cast<const int32_t *>(lds + L.tok);
  pn_schedule<MF>(p.offsets, p.rows, E, offs, mpre, perm, sh_w, sh_c);
  __syncthreads();
  const PnSched S{offs, mpre, perm, E, deal, (int)(blockIdx.x & 7)};
  const int nsl = gridDim.x >> 3;
  const int t_end = pn_walk(S);
  int ct = blockIdx.x >> 3;                // the tile being multiplied
  // two waves of a SIMD (w, w + 4) take different row halves
  const int wm = (w ^ (w >> 2)) & 1, wn = w >> 1;

  // ---- loads.  A line load: 8 rows, lane l brings row l / 8's piece
  // (l % 8) ^ swz (rows 8 (w + 8 j) ..: the XOR depends on w's parity only);
  // a load of W4A16 codes: 32 rows x 32 bytes
  const uint32_t pc = 16u * (uint32_t)((lane & 7) ^ rw_swz(8 * (w & 1) + (lane >> 3)));
  const uint32_t dummy = lds0 + (uint32_t)L.dummy;
  int it = ct, left = 0, ecur = 0, ibuf = 0;
  PnTile itl{}, nx{};
  uint32_t oa[MF], ob[C::NB], os = 0;
  const uint8_t *pa = nullptr, *wb = nullptr, *wsb = nullptr;
  auto tok_dma = [&](const PnTile &tl, int buf) __attribute__((always_inline)) {
    const int32_t *rt = rw_args()->row_token;
    const int wi = pn_fresh_s(w);
    if (rt && wi < MF) {
      const int r = 64 * wi + lane;
      dma4s(uni_ptr(rt), (uint32_t)(tl.row0 + (r < tl.nrows ? r : 0)) * 4u,
            uni(lds0 + (uint32_t)(L.tok + buf * (C::M * 4) + wi * 256)));
    }
  };
  auto src = [&](const int32_t *rt, int r) __attribute__((always_inline)) -> uint32_t {
    if (rt) return (uint32_t)tokb[ibuf * C::M + r];
    return (uint32_t)(itl.row0 + (r < itl.nrows ? r : 0));
  };
  // to tile itl's first stage (its tokens are in LDS), the tokens of the tile
  // after it on their way
  auto bind = [&]() __attribute__((always_inline)) {
    const RwArgPtr q = rw_args();
    const int wi = pn_fresh_s(w), ln = pn_fresh(lane);
    const int64_t er = (int64_t)itl.e * N;
    wb = uni_ptr(q->w_codes + er * kwb);
    pa = uni_ptr(q->a);
    const int32_t *rt = q->row_token;
#pragma unroll
    for (int j = 0; j < MF; ++j)
      oa[j] = src(rt, 8 * (wi + 8 * j) + (ln >> 3)) * (uint32_t)kab + pc;
    if constexpr (FP8) {
#pragma unroll
      for (int j = 0; j < C::NB; ++j)
        ob[j] = (uint32_t)rw_wrow<EPI>(8 * (wi + 8 * j) + (ln >> 3), itl.nt, N) * (uint32_t)kwb + pc;
      const uint32_t db = lds0 + (uint32_t)(L.dec + ibuf * (C::M + PN_N) * 4);
      if (wi < MF) dma4s(uni_ptr(q->a_dec), src(rt, 64 * wi + ln) * 4u, uni(db + wi * 256));
      if (wi >= 4)
        dma4s(uni_ptr(q->w_dec + er), (uint32_t)rw_wrow<EPI>(64 * (wi - 4) + ln, itl.nt, N) * 4u,
              uni(db + C::M * 4 + (wi - 4) * 256));
    } else {
      wsb = uni_ptr(q->w_scales + er * (kwb >> 3));
      ob[0] = (uint32_t)rw_wrow<EPI>(32 * wi + (ln >> 1), itl.nt, N) * (uint32_t)kwb +
              16u * (uint32_t)(ln & 1);
      os = (uint32_t)rw_wrow<EPI>(32 * wi + (ln & 31), itl.nt, N) * (uint32_t)(kwb >> 3);
    }
    left = nst;
    if (it + nsl < t_end) {
      nx = pn_locate<MF>(S, it + nsl, ecur, lane);
      tok_dma(nx, ibuf ^ 1);
    }
  };
  // a stage of loads into the slot at LDS address sb, LPS per wave always
  // (placeholders past the last tile), so that the waits can count
  auto loads = [&](uint32_t sb) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < MF; ++j) dma16s(pa, oa[j], uni(sb + (w + 8 * j) * 1024));
#pragma unroll
    for (int j = 0; j < C::NB; ++j) dma16s(wb, ob[j], uni(sb + C::BOFF + (w + 8 * j) * 1024));
    if constexpr (!FP8) {
      dma4s(wsb, os, uni(sb + C::SOFF + w * 256));
      wsb += 4;
    }
    pa += 128;
    wb += FP8 ? 128 : 32;
  };
  auto issue = [&](uint32_t sb) __attribute__((always_inline)) {
    if (left == 0) {
      it += nsl;
      if (it < t_end) {
        itl = nx;
        ibuf ^= 1;
        bind();
      } else {
        left = 0x7fffffff;
      }
    }
    --left;
    if (it < t_end) {
      loads(sb);
    } else {
      const uint8_t *any = uni_ptr(rw_args()->a);
#pragma unroll
      for (int j = 0; j < C::LPS; ++j) dma4s(any, 0u, uni(dummy));
    }
  };

  if (it < t_end) {
    itl = pn_locate<MF>(S, it, ecur, lane);
    tok_dma(itl, 0);
    wait_vm<0>();
    pn_barrier();
    bind();
    for (int q = 0; q < ns; ++q) {         // ns <= nst: stages of this tile
      --left;
      loads(uni(lds0 + q * C::SLOT));
    }
    pn_wait<C::LPS>(ns - 1);
    pn_barrier();
  }
  int slot = 0, cbuf = 0;
  PnTile cur = itl;
  while (ct < t_end) {
    const int e = cur.e, nt = cur.nt, row0 = cur.row0, nrows = cur.nrows;
    const int nfr = (nrows + 31) >> 5, half = (nfr + 1) >> 1;
    const int fa0 = wm ? half : 0;
    const int mtv = wm ? nfr - half : half;
    const int fb0 = EPI == QD_EPI_SWIGLU ? wn : 2 * wn;
    constexpr int FBS = EPI == QD_EPI_SWIGLU ? 4 : 1;    // the wave's second fragment: fb0 + FBS

    auto run = [&](auto mtv_c) __attribute__((always_inline)) {
      constexpr int MTV = decltype(mtv_c)::value;
      constexpr int MA = MTV > 0 ? MTV : 1;
      constexpr int STEPS = FP8 ? 2 : 4, ITEMS = STEPS * MA;
      constexpr int D = FP8 ? 2 : (MA + 1 < 4 ? MA + 1 : 4);   // A fragments in registers
      constexpr int SYNC = ITEMS - (D - 1);    // in the last step: D - 1 <= MA
      f32x16 acc[MA][2];
#pragma unroll
      for (int i = 0; i < MA; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;
      const int r = lane & 31, h = lane >> 5, sw = rw_swz(r);
      struct AOp {
        uint4 c[FP8 ? 2 : 1];
      };
      const int la = (32 * fa0 + r) * 128;
      // fragment n % MA of step n / MA
      auto rd_a = [&](const unsigned char *sl, int n) __attribute__((always_inline)) -> AOp {
        AOp o;
        const int st = n / MA, i = n % MA;
        if constexpr (FP8) {
#pragma unroll
          for (int k = 0; k < 2; ++k)
            o.c[k] = *reinterpret_cast<const uint4 *>(sl + la + i * 4096 +
                                                      (((4 * st + 2 * h + k) ^ sw) << 4));
        } else {
          o.c[0] = *reinterpret_cast<const uint4 *>(sl + la + i * 4096 + (((2 * st + h) ^ sw) << 4));
        }
        return o;
      };
      // the weights: W4A16 a stage's codes and scales of both fragments, FP8 one
      // step's operands
      struct BOp {
        uint4 c[FP8 ? 4 : 2];
        uint32_t s[2];
      };
      auto rd_b = [&](const unsigned char *sl, int st) __attribute__((always_inline)) -> BOp {
        BOp o;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int f = fb0 + j * FBS;
          if constexpr (FP8) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
              o.c[2 * j + k] = *reinterpret_cast<const uint4 *>(
                  sl + C::BOFF + (32 * f + r) * 128 + (((4 * st + 2 * h + k) ^ sw) << 4));
          } else {
            o.c[j] = *reinterpret_cast<const uint4 *>(sl + C::BOFF + f * 1024 + r * 32 + 16 * h);
            o.s[j] = *reinterpret_cast<const uint32_t *>(sl + C::SOFF + f * 256 + r * 4);
          }
        }
        return o;
      };
      auto sync = [&]() __attribute__((always_inline)) -> uint32_t {
        pn_wait<C::LPS>(ns - 2);
        pn_barrier();
        const uint32_t sb = uni(lds0 + slot * C::SLOT);
        slot = slot + 1 == ns ? 0 : slot + 1;
        return sb;
      };
      AOp a[D];
      BOp b, bn;
      if constexpr (MTV > 0) {
        const unsigned char *sl = lds + slot * C::SLOT;
#pragma unroll
        for (int k = 0; k < D - 1; ++k) a[k] = rd_a(sl, k);
        b = rd_b(sl, 0);
      }
      for (int s = 0; s < nst; ++s) {
        if constexpr (MTV == 0) {
          issue(sync());
        } else {
          const unsigned char *sl = lds + slot * C::SLOT, *sn = sl;
          if constexpr (!FP8) {
            // words 4 h + i of the row's 8 to words 2 st + h (step st)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              const uint4 c = b.c[j];
              const auto e = __builtin_amdgcn_permlane32_swap(c.x, c.y, false, false);
              const auto o = __builtin_amdgcn_permlane32_swap(c.z, c.w, false, false);
              b.c[j] = make_uint4(e[0], o[0], e[1], o[1]);
            }
          }
#pragma unroll
          for (int st = 0; st < STEPS; ++st) {
            if (FP8 && st + 1 < STEPS) bn = rd_b(sl, st + 1);
            bf16x8 bf[2];
            if constexpr (!FP8) {
#pragma unroll
              for (int j = 0; j < 2; ++j) {
                const float sc = (float)scale_pair_of(b.s[j], st >> 1)[st & 1];
                const uint32_t wd = word_of(b.c[j], st);
                const f32x2_pair p0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wd, 256.0f, 0);
                const f32x2_pair p1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wd, 256.0f, 1);
                const f32x2_pair p2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wd, 256.0f, 2);
                const f32x2_pair p3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(wd, 256.0f, 3);
                const f32x8 v = {p0[0] * sc, p0[1] * sc, p1[0] * sc, p1[1] * sc,
                                 p2[0] * sc, p2[1] * sc, p3[0] * sc, p3[1] * sc};
                bf[j] = __builtin_convertvector(v, bf16x8);
              }
            }
#pragma unroll
            for (int i = 0; i < MTV; ++i) {
              const int n = st * MA + i;
              uint32_t sb = 0;
              if (n == SYNC) {
                sb = sync();
                sn = lds + slot * C::SLOT;
                if (s + 1 < nst) bn = rd_b(sn, 0);
              }
              const int m = n + D - 1;
              if (m < ITEMS) a[D - 1] = rd_a(sl, m);
              else if (s + 1 < nst) a[D - 1] = rd_a(sn, m - ITEMS);
              if (n == SYNC) issue(sb);
#pragma unroll
              for (int j = 0; j < 2; ++j) {
                if constexpr (FP8) {
                  struct Two { uint4 x, y; };
                  const v8i av = __builtin_bit_cast(v8i, Two{a[0].c[0], a[0].c[FP8 ? 1 : 0]});
                  const v8i bv = __builtin_bit_cast(v8i, Two{b.c[2 * j], b.c[(2 * j + 1) & (FP8 ? 3 : 1)]});
                  acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                      av, bv, acc[i][j], 0, 0, 0, 127, 0, 127);
                } else {
                  acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                      __builtin_bit_cast(bf16x8, a[0].c[0]), bf[j], acc[i][j], 0, 0, 0);
                }
              }
#pragma unroll
              for (int k = 0; k + 1 < D; ++k) a[k] = a[k + 1];
            }
            if (FP8 || st + 1 == STEPS) b = bn;
          }
        }
      }
      // ---- epilogue: the scales, SwiGLU or plain, bf16 pairs of adjacent
      // columns swapped between neighbouring lanes (4-byte stores)
      if constexpr (MTV > 0) {
        const int ln = pn_fresh(lane), hh = ln >> 5;
        const bool odd = (ln & 1) != 0;
        const int cpair = (ln & 31) & ~1;
        constexpr int NO = EPI == QD_EPI_SWIGLU ? 1 : 2;
        const int ldo = pn_fresh_s(EPI == QD_EPI_SWIGLU ? (N >> 1) : N);
        const float *sa = reinterpret_cast<const float *>(lds + L.dec + cbuf * (C::M + PN_N) * 4);
        const float alpha = FP8 ? 1.0f : rw_args()->w_dec[2 * e + 1];
#pragma unroll
        for (int i = 0; i < MTV; ++i) {
          const int rl = 32 * (fa0 + i) + 4 * hh + (odd ? 1 : 0);
#pragma unroll
          for (int jj = 0; jj < NO; ++jj) {
            const int cb0 = EPI == QD_EPI_SWIGLU ? nt * 128 + 32 * wn : nt * PN_N + 32 * (fb0 + jj);
            if (cb0 >= ldo) continue;
            __builtin_amdgcn_sched_barrier(0);
            unsigned char *ob = reinterpret_cast<unsigned char *>(
                rw_args()->out + (int64_t)(row0 + rl) * ldo + cb0 + cpair);
            float s0 = alpha, s1 = alpha;
            if constexpr (FP8) {
              s0 = sa[C::M + 32 * (fb0 + jj) + (ln & 31)];
              s1 = sa[C::M + 32 * (fb0 + FBS) + (ln & 31)];
            }
            float v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
              float ra = 1.0f;
              if constexpr (FP8) ra = sa[32 * (fa0 + i) + 8 * (q >> 2) + 4 * hh + (q & 3)];
              const float g0 = FP8 ? ra * s0 : s0, g1 = FP8 ? ra * s1 : s1;
              if (EPI == QD_EPI_SWIGLU) {
                const float g = g0 * acc[i][0][q], u = g1 * acc[i][1][q];
                v[q] = FP8 ? rw_swiglu_fp8(g, u) : rw_swiglu_w4a16(g, u);
              } else {
                v[q] = g0 * acc[i][jj][q];
              }
            }
            const bool incol = cb0 + cpair < ldo;
#pragma unroll
            for (int q = 0; q < 16; q += 2) {
              const float send = odd ? v[q] : v[q + 1];
              const float x = __int_as_float(
                  __builtin_amdgcn_mov_dpp(__float_as_int(send), 0xB1, 0xF, 0xF, false));
              const f32x2_t pr = odd ? f32x2_t{x, v[q + 1]} : f32x2_t{v[q], x};
              const uint32_t pk = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2_t));
              const int qr = 8 * (q >> 2) + (q & 3);
              if (incol && rl + qr < nrows)
                *reinterpret_cast<uint32_t *>(ob + (size_t)qr * ldo * 2) = pk;
            }
          }
        }
        // the stores' lane branches join here, so that they do not make the
        // scalar state of the tile loop look divergent to the compiler
        asm volatile("" ::: "memory");
      }
    };
    auto pick = [&](auto self, auto n_c) __attribute__((always_inline)) {
      constexpr int n = decltype(n_c)::value;
      if constexpr (n == 0) {
        run(std::integral_constant<int, 0>{});
      } else {
        if (mtv == n) run(std::integral_constant<int, n>{});
        else self(self, std::integral_constant<int, n - 1>{});
      }
    };
    pick(pick, std::integral_constant<int, MF>{});
    // the issue cursor is ns (<= nst) stages ahead: at the next tile
    ct += nsl;
    cur = itl;
    cbuf ^= 1;
  }
  wait_vm<0>();
}

// A tile's fixed time, in that of a 32-row fragment.  Over 225 GEMMs each (1 to 128
// experts of 1 to 2048 rows, K 384 to 4096, N 768 to 8192) the height is 0.5% (FP8) and
// 0.7% (W4A16) from the best on average.  With 2 for both and without the spread of the
// tiles' number it was 0.9 and 1.3%: FP8, 8 experts of 256 rows, K = 4096, N = 3072:
// 78 us on 128-row tiles, 43 on 192.
constexpr double RW_TILE_FP8 = 2.0, RW_TILE_W4A16 = 7.0;

struct RowsPlan {
  bool ok;
  int mf, ns, grid, lds;
  PnDeal deal;
  double time;               // estimated, in that of a 32-row fragment
};

// for whole stages, two of them or more, and operands that 32-bit byte offsets
// reach (a_rows: rows of the activations)
inline RowsPlan rows_plan(bool fp8, int64_t rows, int64_t a_rows, int E, int64_t N, int64_t K,
                          int epilogue) {
  RowsPlan pl{};
  const int64_t kab = fp8 ? K : 2 * K, kwb = fp8 ? K : K / 2;
  const int64_t lim = 1LL << 32;
  if (kab < 256 || kab % 128 != 0 || N % 32 != 0 || E > PN_EMAX) return pl;
  if ((std::max(a_rows, rows) + 1) * kab >= lim || N * kwb >= lim || rows * 4 >= lim) return pl;
  const int nst = (int)(kab / 128);
  const int ntn = epilogue == QD_EPI_SWIGLU ? (int)((N / 2 + 127) / 128) : (int)((N + PN_N - 1) / PN_N);
  const PnHeight h = pn_height(rows, E, ntn, fp8 ? RW_TILE_FP8 : RW_TILE_W4A16, true, false, [&](int mf) {
    int ns = std::min(5, nst);
    while (ns >= 2 && rw_layout(fp8, mf, ns, E).total > PN_LDS_MAX) --ns;
    return ns;
  });
  if (h.mf == 0) return pl;
  pl.mf = h.mf;
  pl.ns = h.ns;
  pl.time = h.time;
  pl.lds = rw_layout(fp8, h.mf, h.ns, E).total;
  pl.grid = (int)std::min<int64_t>(256, qdt::tile_grid(rows, E, 64 * pl.mf, ntn));
  pl.deal = pn_deal(h, ntn, pl.grid);
  pl.ok = true;
  return pl;
}

template <bool FP8, int MF, int EPI>
void launch_rows_one(const RowsArgs &p, const RowsPlan &pl, hipStream_t s) {
  auto kern = gemm_rows_kernel<FP8, MF, EPI>;
  static const bool attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               PN_LDS_MAX) == hipSuccess;
  (void)attr;
  hipLaunchKernelGGL(kern, dim3((unsigned)pl.grid), dim3(PN_THREADS), (size_t)pl.lds, s, p, pl.deal,
                     pl.ns);
}
template <bool FP8, int EPI>
void launch_rows_epi(const RowsArgs &p, const RowsPlan &pl, hipStream_t s) {
  switch (pl.mf) {
    case 5: launch_rows_one<FP8, 5, EPI>(p, pl, s); break;
    case 3: launch_rows_one<FP8, 3, EPI>(p, pl, s); break;
    case 2: launch_rows_one<FP8, 2, EPI>(p, pl, s); break;
    default: launch_rows_one<FP8, 1, EPI>(p, pl, s); break;
  }
}
template <bool FP8>
void launch_rows(const RowsArgs &p, int epi, const RowsPlan &pl, hipStream_t s) {
  if (epi == QD_EPI_SWIGLU) launch_rows_epi<FP8, QD_EPI_SWIGLU>(p, pl, s);
  else launch_rows_epi<FP8, QD_EPI_NONE>(p, pl, s);
}

}  // namespace qdr
