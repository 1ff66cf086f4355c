// Grouped W4A4 GEMM for a handful of rows.
//
// With few rows the work is the weights of the few experts they touch (14 MB
// for one token on eight experts at K = 2048, 1536 weight rows), and the
// decode kernel's blocks of 256 weight rows are too coarse for it: 48 of them,
// on 256 CUs, each walking all of K behind a barrier per 256 elements.  Here a
// wave takes 32 weight rows (SwiGLU: 16 gate rows and the matching 16 up rows)
// of one expert and streams them over its part of K through an LDS ring of its
// own (direct global->LDS loads of whole 128-byte lines, as in the decode
// kernel), with no barrier before the sum; up to four waves share a block's K,
// and their partial sums meet in LDS and are added in wave order, so the
// result is deterministic.  Each wave decodes the activation rows (8 per pass)
// itself: with few rows that is cheaper than meeting the others.
//
// Bound: latency (launch, offsets, tokens, one or two trips to HBM, the sum)
// for one token, HBM with operand decode beside it for more.  Loads straight
// to registers in fragment order were tried first: 16 rows 2 KB apart in every
// quarter wave made them 64 line accesses per load, and one token's W13 took
// 14.2 us instead of 10.4.
//
// Fragment layout (16x16x32 MFMA): lane l holds row l % 16 of a 16-row
// fragment, elements 64 (l / 16) .. + 63 of a 256-element chunk; k-step
// (c, s) takes elements 32 c + 8 s .. + 7 of them, for A and B alike.
#include "gemm_few.h"
#include "lds_dma.h"

namespace qdf {

using namespace qd;
using namespace qdg;
using qdl::uni;

namespace {

__device__ __forceinline__ f32x4 mfma16(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// one lane's 64 elements of a row in a chunk
struct Frag {
  uint4 c0, c1;
  uint32_t s;
};

__device__ __forceinline__ f16x8 frag_step(const Frag &f, int c, int s) {
  return decode8_sel(word_of(c ? f.c1 : f.c0, s), scale_pair_of(f.s, c), s >= 2);
}

// a wave's LDS stage: weight codes of 32 rows (128 bytes each, 16-byte piece q
// of row r at 128 r + 16 (q ^ r % 8)), their scale dwords in lane order, then
// the activation's (and the residual's) 8 rows the same way
constexpr int FW_XR = 8;                 // activation rows per pass
constexpr int FW_X = 4096 + 512;
constexpr int FW_XBYTES = FW_XR * 128 + 256;

template <bool RAC, int EPI>
__global__ __launch_bounds__(64 * FW_WAVES) void gemm_few_kernel(GemmArgs p, int nblk, int ngrp,
                                                                 int lsplit) {
  constexpr int D = RAC ? 2 : 3;         // stages in flight per wave
  constexpr int ST = FW_X + (RAC ? 2 : 1) * FW_XBYTES;
  constexpr int LX = RAC ? 4 : 2, LPS = 6 + LX;   // loads of a stage: activations, all
  __shared__ __align__(16) unsigned char ring[FW_WAVES][D][ST];
  __shared__ float red[16];
  const int tid = threadIdx.x, lane = tid & 63, w = (int)uni((uint32_t)tid >> 6);
  const int lr = lane & 15, g = lane >> 4;
  const int K = p.K, N = p.N;
  const int kb2 = K >> 1, kb16 = K >> 4;
  const int split = 1 << lsplit, kp = w & (split - 1);
  // the workgroup's expert: the a-th one that has rows
  int a = (int)uni(blockIdx.x / (uint32_t)ngrp), e = -1, row0 = 0, rows = 0;
  const int nb = (int)(blockIdx.x - a * ngrp) * (FW_WAVES >> lsplit) + (w >> lsplit);
  if (!p.offsets) {
    if (a == 0) e = 0;
    rows = (int)p.rows;
  } else {
    // lane l: experts e0 + 2 l and the next
    for (int e0 = 0; e0 < p.E; e0 += 128) {
      const int x = e0 + 2 * lane;
      int o[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) o[q] = p.offsets[min(x + q, p.E)];
      const uint64_t m0 = __ballot(o[1] > o[0]), m1 = __ballot(o[2] > o[1]);
      const int n = __popcll(m0) + __popcll(m1);
      if (a < n) {
        const uint64_t lt = (1ull << lane) - 1ull;
        const int rk = __popcll(m0 & lt) + __popcll(m1 & lt);
        const bool h0 = o[1] > o[0] && rk == a;
        const bool h1 = o[2] > o[1] && rk + (o[1] > o[0]) == a;
        const int src = __ffsll((unsigned long long)__ballot(h0 || h1)) - 1;
        const bool odd = (__ballot(h1) >> src) & 1ull;
        e = e0 + 2 * src + (odd ? 1 : 0);
        row0 = __builtin_amdgcn_readlane(odd ? o[1] : o[0], src);
        rows = __builtin_amdgcn_readlane(odd ? o[2] : o[1], src) - row0;
        break;
      }
      a -= n;
    }
  }
  float vmax = 0.0f;
  if (e >= 0) {
    // the wave's two weight fragments (a block past the last one reads the
    // last and stores nothing)
    const bool live = nb < nblk;
    const int bk = live ? nb : nblk - 1;
    const int I = N >> 1;
    const int n0 = EPI == QD_EPI_SWIGLU ? 16 * bk : FW_N * bk;
    const int n1 = EPI == QD_EPI_SWIGLU ? I + 16 * bk : FW_N * bk + 16;
    const int64_t r0 = (int64_t)e * N + n0, r1 = (int64_t)e * N + n1;
    const uint8_t *wc[2] = {p.w_codes + r0 * kb2, p.w_codes + r1 * kb2};
    const bool sfrag = p.w_sfrag != nullptr;
    const int64_t nc = K >> 8;
    const uint8_t *ws[2] = {sfrag ? p.w_sfrag + (r0 >> 4) * nc * 256 : p.w_scales + r0 * kb16,
                            sfrag ? p.w_sfrag + (r1 >> 4) * nc * 256 : p.w_scales + r1 * kb16};
    const int nch = (K + 255) >> 8;
    const int nmy = kp < nch ? (nch - kp + split - 1) >> lsplit : 0;   // chunks kp, kp + split, ..
    const float sw = p.w_gs[2 * e + 1];
    const float alpha = p.a_gs[1] * sw, alpha_r = RAC ? p.r_gs[1] * sw : 0.0f;
    // direct global->LDS loads: code load i of a fragment brings 8 rows of 128
    // bytes, lane l row 8 i + l / 8, piece (l % 8) ^ (l / 8); pieces past K
    // (its last chunk) repeat the row's first piece, and the scales of their
    // elements count as zero
    const uint32_t lds0 = (uint32_t)(uintptr_t)&ring[w][0][0];
    const int pr = lane >> 3, pq = (lane & 7) ^ pr;
    const int b0 = 128 * lr + 16 * ((2 * g) ^ (lr & 7));
    const int xr = lr & (FW_XR - 1);
    const int x0 = FW_X + 128 * xr + 16 * ((2 * g) ^ xr);
    for (int p0 = 0; p0 < rows; p0 += FW_XR) {
      const int nrow = min(FW_XR, rows - p0);
      // the pass's tokens by scalar loads, which the vector loads' order does
      // not hold up
      int tok = 0;
#pragma unroll
      for (int q = 0; q < FW_XR; ++q) {
        const int gr = row0 + p0 + min(q, nrow - 1);
        const int t = p.row_token ? p.row_token[gr] : gr;
        tok = pr == q ? t : tok;
      }
      const int toks = __shfl(tok, 8 * ((lane >> 2) & (FW_XR - 1)), 64);
      auto issue_w = [&](int i, int slot) __attribute__((always_inline)) {
        const int ch = kp + (min(i, nmy - 1) << lsplit);
        const uint32_t sb = uni(lds0 + slot * ST);
        const uint32_t po = (uint32_t)(ch * 128 + (ch * 256 + 32 * pq < K ? 16 * pq : 0));
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          qdl::dma16s(qdl::uni_ptr(wc[j]), (uint32_t)(pr * kb2) + po, sb + 2048 * j);
          qdl::dma16s(qdl::uni_ptr(wc[j]), (uint32_t)((pr + 8) * kb2) + po, sb + 2048 * j + 1024);
        }
        const uint32_t so = sfrag ? (uint32_t)(ch * 256 + lane * 4)
                                  : (uint32_t)(lr * kb16 + ch * 16 + (ch * 256 + 64 * g < K ? 4 * g : 0));
#pragma unroll
        for (int j = 0; j < 2; ++j) qdl::dma4s(qdl::uni_ptr(ws[j]), so, sb + 4096 + 256 * j);
      };
      auto issue_x = [&](int i, int slot) __attribute__((always_inline)) {
        const int ch = kp + (min(i, nmy - 1) << lsplit);
        const uint32_t sb = uni(lds0 + slot * ST + FW_X);
        const int co = ch * 128 + (ch * 256 + 32 * pq < K ? 16 * pq : 0);
        const int so = ch * 16 + (ch * 256 + 64 * (lane & 3) < K ? 4 * (lane & 3) : 0);
        qdl::dma16(p.a_codes + (int64_t)tok * kb2 + co, sb);
        qdl::dma4(p.a_scales + (int64_t)toks * kb16 + so, sb + FW_XR * 128);
        if (RAC) {
          qdl::dma16(p.r_codes + (int64_t)tok * kb2 + co, sb + FW_XBYTES);
          qdl::dma4(p.r_scales + (int64_t)toks * kb16 + so, sb + FW_XBYTES + FW_XR * 128);
        }
      };
      f32x4 acc[2], accr[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[j] = accr[j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (nmy > 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) issue_w(d, d);
#pragma unroll
        for (int d = 0; d < D; ++d) issue_x(d, d);
        int slot = 0;
        // (one chunk's code in a rolled loop: straight-line code that runs
        // once is fetched at memory latency)
#pragma unroll 1
        for (int i = 0; i < nmy; ++i) {
          // the loads issued after this stage's: the activations of the
          // stages the prologue began, all of the later ones
          if (i == 0) qdl::wait_vm<(D - 1) * LX>();
          else if (D > 2 && i == 1) qdl::wait_vm<LX + LPS>();
          else qdl::wait_vm<(D - 1) * LPS>();
          const unsigned char *sl = &ring[w][slot][0];
          const bool in = (kp + (i << lsplit)) * 256 + 64 * g < K;
          Frag f[2], x, r{};
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            f[j].c0 = *reinterpret_cast<const uint4 *>(sl + 2048 * j + b0);
            f[j].c1 = *reinterpret_cast<const uint4 *>(sl + 2048 * j + (b0 ^ 16));
            f[j].s = *reinterpret_cast<const uint32_t *>(sl + 4096 + 256 * j + lane * 4);
            f[j].s = in ? f[j].s : 0u;
          }
          auto rd = [&](Frag &o, const unsigned char *q) __attribute__((always_inline)) {
            o.c0 = *reinterpret_cast<const uint4 *>(q + x0);
            o.c1 = *reinterpret_cast<const uint4 *>(q + (x0 ^ 16));
            o.s = *reinterpret_cast<const uint32_t *>(q + FW_X + FW_XR * 128 + 16 * xr + 4 * g);
          };
          rd(x, sl);
          if (RAC) rd(r, sl + FW_XBYTES);
          qdl::wait_lds();               // the slot may be refilled
          issue_w(i + D, slot);
          issue_x(i + D, slot);
          slot = slot + 1 == D ? 0 : slot + 1;
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
              const f16x8 f0 = frag_step(f[0], c, s), f1 = frag_step(f[1], c, s);
              const f16x8 xa = frag_step(x, c, s);
              acc[0] = mfma16(xa, f0, acc[0]);
              acc[1] = mfma16(xa, f1, acc[1]);
              if (RAC) {
                const f16x8 ra = frag_step(r, c, s);
                accr[0] = mfma16(ra, f0, accr[0]);
                accr[1] = mfma16(ra, f1, accr[1]);
              }
            }
        }
        qdl::wait_vm<0>();               // the loads past the last stage
      }
      if (split > 1) {
        // the split's sums in wave order, by its first wave (each wave's in
        // its own ring, whose loads are done)
        f32x4 *part = reinterpret_cast<f32x4 *>(&ring[w][0][0]);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          part[64 * j + lane] = acc[j];
          if (RAC) part[64 * (2 + j) + lane] = accr[j];
        }
        __syncthreads();
        if (kp == 0) {
          for (int ww = 1; ww < split; ++ww) {
            const f32x4 *q = reinterpret_cast<const f32x4 *>(&ring[w + ww][0][0]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              acc[j] += q[64 * j + lane];
              if (RAC) accr[j] += q[64 * (2 + j) + lane];
            }
          }
        }
      }
      if (kp == 0 && live) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int rl = 4 * g + q;
          if (rl >= nrow) continue;
          const int64_t row = row0 + p0 + rl;
          float v[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            v[j] = alpha * acc[j][q];
            if (RAC) v[j] = v[j] - alpha_r * accr[j][q];
          }
          if (EPI == QD_EPI_SWIGLU) {
            const float hv = v[0] / (1.0f + expf(-v[0])) * v[1];
            const uint32_t hb = f32_to_bf16_bits(hv);
            p.out[row * I + n0 + lr] = (uint16_t)hb;
            vmax = fmaxf(vmax, fabsf(bf16_bits_to_f32(hb)));
          } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              const uint32_t hb = f32_to_bf16_bits(v[j]);
              p.out[row * N + (j ? n1 : n0) + lr] = (uint16_t)hb;
              vmax = fmaxf(vmax, fabsf(bf16_bits_to_f32(hb)));
            }
          }
        }
      }
      if (split > 1 && p0 + FW_XR < rows) __syncthreads();   // the sums are read first
    }
  }
  if (RAC && p.r_bitmap && blockIdx.x == 0 && w == 0) {
    // S in ascending order from the bitmap (<= 128 words: two per lane)
    const int nwd = K >> 5;
    uint32_t m0 = 2 * lane < nwd ? p.r_bitmap[2 * lane] : 0u;
    uint32_t m1 = 2 * lane + 1 < nwd ? p.r_bitmap[2 * lane + 1] : 0u;
    const int c = __popc(m0) + __popc(m1);
    int xs = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(xs, o, 64);
      if (lane >= o) xs += y;
    }
    int pos = xs - c;
    while (m0) {
      p.sel_out[pos++] = 64 * lane + (__ffs(m0) - 1);
      m0 &= m0 - 1u;
    }
    while (m1) {
      p.sel_out[pos++] = 64 * lane + 32 + (__ffs(m1) - 1);
      m1 &= m1 - 1u;
    }
  }
  const float m = block_max(vmax, red);
  put_amax(p, m);
}

}  // namespace

// Where this kernel is the faster one.  It streams an expert's weights once per
// 8 rows, the decode kernel once per 48, the panel kernel once; p is the number of
// passes an average expert with rows takes (half a pass more than the mean once
// the rows of an expert vary).
//
//  * K a multiple of 256, against the decode kernel, which hands blocks of 256
//    weight rows of the experts with rows to 256 CUs (u of them, if every row has
//    an expert of its own) and takes the time of whole rounds of the chip.  Few
//    blocks leave most of it idle: u * p up to 96, with the residual or K below
//    1024 up to 128, and at most four passes (two and a half below 1024, where a
//    pass is mostly its fixed part).  K = 2048, 1536 weight rows, one expert: 16
//    rows 13.8 against 20.4 us, 32 rows 20.3 against 21.9, 48 rows 26.4 against
//    21.8; K = 4096, 12288 rows on two experts of 16 rows 52.0 against 34.3; one
//    token on eight experts (u = 48) 10.4 against 20.8.  (Here and below weights
//    that no cache holds, except for the token.)
//  * Above the decode kernel's 48 rows per expert, against the tile and panel
//    kernels: one or two experts of K >= 2048 and a few blocks each, up to 64 rows
//    (two experts of 64, K = 4096, N = 3072: 43 against 55 us, with K_s = 128 50
//    against 55, K / 2 50 against 88; one of 64, K = 2048, N = 1536: 27 against 32,
//    with K_s = 64 30 either way; K = 1536, N = 4096: 64 rows 36 either way).
//  * With the residual also u >= 320 (a second round with few units in it) at up
//    to four rows per expert: K = 4096, N = 12288, 8 experts: 3 rows each 91
//    against 98, 12 rows each 122 against 98; 128 experts with one row, N = 3072:
//    83 against 96.  Without the residual the decode kernel keeps these.
//  * Other K: up to four passes against the panel kernel where it takes them (K =
//    384, N = 2048, one expert: 24 rows 14.1 against 15.1, 48 rows 20.5 against
//    16.4); against the generic kernel two and a half for K of 1024 and more (K =
//    2112, N = 2048: 64 rows on 4 experts 21.2 against 26.3, 128 rows 29.0
//    against 26.4), below one, with the residual one and a half (K = 320: 128 rows
//    on 16 experts 14.4 against 12.0, with it 14.6 against 15.1).
constexpr int64_t kFewRows = 128;
constexpr int64_t kFewSecond = 320;
constexpr int64_t kBitmapKMax = 4096;    // two bitmap words per lane of one wave
constexpr int64_t kFewWaves = 4096;      // waves that fill the chip's queues

FwPlan few_plan(int64_t rows, int E, int64_t N, int64_t K, int Ks, int epilogue, bool bitmap) {
  FwPlan pl{};
  if (rows > kFewRows || E > 1024 || K % 64 != 0 || K > 0x7fffff || N % 32 != 0) return pl;
  if (bitmap && (Ks <= 0 || K > kBitmapKMax)) return pl;
  const int64_t nblk = epilogue == QD_EPI_SWIGLU ? N / 2 / 16 : N / FW_N;
  const int64_t act = std::min<int64_t>(std::max<int64_t>(rows, 1), E);   // experts with rows
  const int64_t u = act * ((N + 255) / 256);
  // eight times p
  const int64_t p8 = E == 1 ? (rows + 7) / 8 * 8 : std::max<int64_t>(8, rows / act + 4);
  if (K % 256 == 0) {
    const bool brief = K < 1024;
    const bool idle = p8 <= (brief ? 20 : 32) && u * p8 <= 8 * (Ks > 0 || brief ? 128 : 96);
    const bool dense = rows > 48 * (int64_t)E && K >= 2048 && u <= 24 && p8 <= 68;
    if (!idle && !dense && !(Ks > 0 && u >= kFewSecond && rows <= 4 * act)) return pl;
  } else {
    const bool panel = K >= 256 && K % 128 == 0 && N % 128 == 0;
    if (p8 > (panel ? 32 : K >= 1024 ? 20 : Ks > 0 ? 12 : 9)) return pl;
  }
  // split K over waves while a wave per block would leave the chip short of
  // waves in flight
  int ls = 0;
  while (ls < 2 && (K + 255) / 256 >= (2 << ls) && act * nblk << ls < kFewWaves) ++ls;
  const int per = FW_WAVES >> ls;
  pl.split = ls;
  pl.nblk = (int)nblk;
  pl.ngrp = (int)((nblk + per - 1) / per);
  if (act * pl.ngrp > 0x7fffffffLL) return pl;
  pl.grid = (int)(act * pl.ngrp);
  pl.ok = true;
  return pl;
}

void launch_few(const GemmArgs &p, int epilogue, const FwPlan &pl, hipStream_t s) {
  const dim3 grid((unsigned)pl.grid), block(64 * FW_WAVES);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, 0, s, p, pl.nblk, pl.ngrp, pl.split);
  };
  if (p.Ks > 0) {
    if (epilogue == QD_EPI_SWIGLU) go(gemm_few_kernel<true, QD_EPI_SWIGLU>);
    else go(gemm_few_kernel<true, QD_EPI_NONE>);
  } else {
    if (epilogue == QD_EPI_SWIGLU) go(gemm_few_kernel<false, QD_EPI_SWIGLU>);
    else go(gemm_few_kernel<false, QD_EPI_NONE>);
  }
}

}  // namespace qdf
