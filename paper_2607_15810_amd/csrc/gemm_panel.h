// Grouped W4A4 GEMM for tens of rows per expert and more (gemm_panel_kernel).
// The compiled sizes live in gemm_panel_<MF>.hip, the choice among them in
// gemm.hip.
//
//  * Workgroup tile: up to 64 MF rows of one expert x 256 weight rows
//    (SwiGLU: 128 gate rows and the matching 128 up rows), eight waves in a
//    2 x 4 grid, each up to 32 MF rows x 64 weight rows on
//    v_mfma_f32_32x32x16_f16.  Two waves share each SIMD, so one wave's
//    operand decode runs under the other's MFMAs; the row halves alternate
//    between the two waves of a SIMD, so a tile with an odd number of 32-row
//    fragments loads the SIMDs evenly.
//  * M-tiles never straddle experts.  An expert of f 32-row fragments is cut
//    into ceil(f / 2 MF) tiles of equal height (to one fragment): a remainder
//    of a few rows costs the fragments it has, not a second pass over the
//    weights with nearly empty tiles.
//  * Persistent: one workgroup per CU (two with short rings of 64-row tiles)
//    walks a static list of tiles, experts of tall tiles first, so that the last,
//    partial round of the chip holds the smallest ones.  An M-tile's weight-row tiles (and the M-tiles of an expert
//    that has several) go to one XCD, where they share activation rows (and
//    weights) in its L2.  The stages of all its tiles form one stream through an
//    LDS ring of NS slots, so the loads of the next tile run under the end of this
//    one.  (At 320 rows the kernel spills nine registers, 40 bytes of scratch per
//    lane; their reload before the epilogue waits for the loads in flight too, so
//    there they run under the last stages but not under the epilogue.)
//  * A stage is 128 K-elements of the tile's rows, codes and scales of both
//    operands, filled by direct global->LDS loads (16 rows x 64 contiguous
//    bytes each, the 16-byte pieces of a row placed by a row-dependent XOR, so
//    the fragment reads are free of bank conflicts).  One barrier per stage,
//    just before its last fragment is multiplied: every operand of the stage
//    is in registers then, so the slot is refilled at once and the first
//    operands of the next stage are read under the last fragment's MFMAs.
//  * Inside a stage lane (row r, half h) owns elements 64 h .. 64 h + 63;
//    MFMA k-step s (0..7) takes elements 8 s .. 8 s + 7 of each half, for A
//    and B alike (a common permutation of K).
//  * RAC, compact form: while a stage is in LDS the workgroup copies the
//    selected channels of its weight rows out of it, decoded to f16, into a
//    [256 rows][K_s] table; after the K loop the accumulators are rescaled by
//    -s_dec_x / s_dec_r and the residual (f16, compacted per token) is
//    multiplied onto them against that table in stages of 32 channels that
//    ride the same ring, so the epilogue's single scale -s_dec_r * s_dec_w
//    yields s_dec_x s_dec_w acc - s_dec_r s_dec_w accr with one extra f32
//    rounding of the main sum.  Dense form (no table): a second pass over K
//    with the masked residual as the A operand, after the same rescale.
//
// What bounds it: for hundreds of rows per expert the operand decode and the
// MFMAs of two waves per SIMD (K = 4096, 256 +- 16 rows on each of 128
// experts, 3072 weight rows, K_s = 128: 0.90 ms = 0.92 PFLOP/s; 0.73 ms with
// the refills left out, 0.47 ms with decode and MFMAs left out).  Tile heights
// of up to 320 rows in steps of 32 are what it was built for: a kernel of
// 256 x 128 tiles with the residual took 1.08 ms there, one of 256 x 256
// tiles without the residual 0.92 ms against 0.82 ms here, as every expert
// with 257 rows or more paid a second, nearly empty tile.  With skewed routing
// (popularity rank^-1.2) the sorted walk is what counts: K = 2048, 4000 tokens,
// W13 319 -> 291 us, 1000 tokens 152 -> 137 us against one in expert order.
#pragma once
#include "gemm_args.h"
#include "lds_dma.h"
#include "panel_sched.h"

namespace qdp {

using namespace qd;
using namespace qdl;
using qdg::GemmArgs;
using qdg::bf16x2_t;
using qdg::f32x16;
using qdg::f32x2_t;
using qdg::mfma32;
using qdg::swiglu_fast;
using qdg::word_of;

constexpr int PN_K = 128;
constexpr int PN_PAD = 4;                // f16 columns past each compact table row

template <int MF>
struct PnCfg {
  static constexpr int M = 64 * MF;
  // slot: A codes [M / 16 row groups][1 KB], A scales [M][8 B], B codes
  // [16 row groups][1 KB], B scales [16 row groups][128 B]
  static constexpr int ASCL = M * 64;
  static constexpr int BCODE = M * 72;
  static constexpr int BSCL = M * 72 + 16384;
  static constexpr int SLOT = M * 72 + 18432;
  static constexpr int NA = 6 * MF;            // A loads of a stage: 4 MF codes, 2 MF scales
  static constexpr int NJ = (NA + 7) / 8;      // of them per wave
  static constexpr int LPS = 3 + NJ;           // loads per wave and stage
};

struct PnLayout {
  int tab, sel, tok, dummy, offs, mpre, perm, total;
};

// after the ring: the compact table and S (RAC, compact form), the tokens of
// two tiles, the target of placeholder loads, the tile schedule
__host__ __device__ inline PnLayout pn_layout(int mf, int ns, int ksa, int E) {
  PnLayout L{};
  int o = ns * (64 * mf * 72 + 18432);
  auto take = [&](int bytes) { const int at = o; o += (bytes + 15) & ~15; return at; };
  L.tab = take(ksa ? PN_N * (ksa + PN_PAD) * 2 : 0);
  L.sel = take(ksa * 4);
  L.tok = take(2 * 64 * mf * 4);
  L.dummy = take(1024);
  L.offs = take((E + 1) * 4);
  L.mpre = take((E + 1) * 4);
  L.perm = take(E * 2);
  L.total = o;
  return L;
}

// 16-byte piece p of tile row ri (0..15 within a 16-row load) sits at piece
// p ^ pn_swz(ri) of the row's 64-byte LDS record
__device__ __forceinline__ int pn_swz(int ri) { return ((ri >> 1) ^ (ri >> 2)) & 3; }

// the kernel's arguments read anew from the kernarg segment (GemmArgs is the
// kernel's first parameter): those the K loop seldom needs hold no scalar
// registers across it
typedef const __attribute__((address_space(4))) GemmArgs *PnArgPtr;
__device__ __forceinline__ PnArgPtr pn_args() {
  PnArgPtr q = (PnArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(q));
  return q;
}

// the tile's 32-row weight fragment f (0..7) starts at this weight row (0 for
// a fragment wholly past N: any valid rows, never stored); SwiGLU: fragments
// 0..3 gate rows, 4..7 the matching up rows
template <int EPI>
__device__ __forceinline__ int pn_wrow(int f, int nt, int N) {
  if (EPI == QD_EPI_SWIGLU) {
    const int I = N >> 1, c = nt * 128 + 32 * (f & 3);
    return c < I ? c + (f < 4 ? 0 : I) : 0;
  }
  const int c = nt * PN_N + 32 * f;
  return c < N ? c : 0;
}

template <int MF, int EPI>
__global__ __launch_bounds__(PN_THREADS, MF == 1 ? 4 : 2) void gemm_panel_kernel(
    GemmArgs p, PnDeal deal, int ns, int dense) {
  using C = PnCfg<MF>;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ int sh_w[8];
  __shared__ int sh_c[8][2 * MF + 1];
  __shared__ float red[16];
  const int tid = threadIdx.x, lane = tid & 63, w = (int)uni((uint32_t)tid >> 6);
  const int K = p.K, N = p.N, E = p.E;
  const int kb2 = K >> 1, kb16 = K >> 4;
  const int nst = K / PN_K;
  const bool cmp = p.Ks > 0 && !dense;      // compact residual
  const int ksa = cmp ? p.ksa : 0, ksp = ksa + PN_PAD;
  const PnLayout L = pn_layout(MF, ns, ksa, E);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  int32_t *offs = reinterpret_cast<int32_t *>(lds + L.offs);
  int32_t *mpre = reinterpret_cast<int32_t *>(lds + L.mpre);
  int32_t *sel_l = reinterpret_cast<int32_t *>(lds + L.sel);
  const int32_t *tokb = reinterpret_cast<const int32_t *>(lds + L.tok);

  uint16_t *perm = reinterpret_cast<uint16_t *>(lds + L.perm);
  pn_schedule<MF>(p.offsets, p.rows, E, offs, mpre, perm, sh_w, sh_c);
  const bool per_expert = p.sel_stride != 0;
  if (cmp) {
    if (!per_expert)
      for (int i = tid; i < ksa; i += PN_THREADS) sel_l[i] = i < p.Ks ? p.sel[i] : 0;
    // pad columns of the compact table are zero (the residual's are too)
    const int pad = ksa - p.Ks;
    for (int i = tid; i < PN_N * pad; i += PN_THREADS)
      *reinterpret_cast<_Float16 *>(lds + L.tab + ((i / pad) * ksp + p.Ks + i % pad) * 2) =
          (_Float16)0.0f;
  }
  // acc -> acc * inv_c + accr, then the scale -s_dec_r * s_dec_w.  A residual
  // whose tensor scale is below 2^-60 of the activation's is left out (its
  // share of any output is far below f32 resolution).
  const float a_dec = p.a_gs[1];
  float inv_c = 0.0f, t_dec = a_dec;
  bool res_on = false;
  if (p.Ks > 0) {
    const float r_dec = p.r_gs[1];
    inv_c = -(a_dec / r_dec);
    res_on = r_dec > 0.0f && fabsf(inv_c) <= 0x1p60f;
    if (res_on) t_dec = -r_dec;
  }
  res_on = uni((uint32_t)res_on) != 0u;
  const int nmain = res_on && dense ? 2 * nst : nst;
  const int nres = res_on && cmp ? (ksa + 31) >> 5 : 0;
  __syncthreads();
  const PnSched S{offs, mpre, perm, E, deal, (int)(blockIdx.x & 7)};
  const int nsl = gridDim.x >> 3;
  const int t_end = pn_walk(S);            // tiles of this XCD's walk
  int ct = blockIdx.x >> 3;                // the tile being multiplied
  float vmax = 0.0f;

  // two waves of a SIMD (w, w + 4) take different row halves
  const int wm = (w ^ (w >> 2)) & 1, wn = w >> 1;
  const int ri = lane >> 2;
  const int pcs = (lane & 3) ^ pn_swz(ri);
  const uint32_t pc = 16u * (uint32_t)pcs;
  // ---- loads.  A 16-row load of codes: lane l brings row l / 4's piece
  // (l % 4) ^ swz; a scale load: 32 rows, lane l the dword of row / half as
  // the slot stores it
  const bool sfrag = p.w_sfrag != nullptr;
  const uint32_t ob = (uint32_t)ri * (uint32_t)kb2 + pc;
  const uint32_t obs = sfrag ? (uint32_t)((lane >> 5) * (K >> 8) * 256 + (lane & 31) * 4)
                             : (uint32_t)((16 * (lane >> 5) + (lane & 15)) * kb16 +
                                          4 * ((lane >> 4) & 1));
  const int bstep = sfrag ? 128 : 8;
  const uint32_t ring = lds0;
  const uint32_t dummy = lds0 + (uint32_t)L.dummy;
  // the issue cursor: `left` stages of its tile's current phase (0 the
  // activations, 1 the dense residual's pass, 2 the compact residual's
  // stages, 3 no tile left), and this wave's source pointers of the next one
  int it = ct, left = 0, phase = 0, ecur = 0, ibuf = 0;
  PnTile itl{}, nx{};                          // its tile and the one after
  uint32_t oa[C::NJ];
  const uint8_t *pa = nullptr, *ps = nullptr, *wb[2] = {}, *wsb = nullptr;
  auto tok_dma = [&](const PnTile &tl, int buf) __attribute__((always_inline)) {
    const int32_t *rt = pn_args()->row_token;
    const int wi = pn_fresh_s(w);
    if (rt && wi < MF) {
      const int r = 64 * wi + lane;
      dma4s(uni_ptr(rt), (uint32_t)(tl.row0 + (r < tl.nrows ? r : 0)) * 4u,
            uni(lds0 + (uint32_t)(L.tok + buf * (C::M * 4) + wi * 256)));
    }
  };
  // source row of tile row r of the issue cursor's tile
  auto src = [&](const int32_t *rt, int r) __attribute__((always_inline)) -> uint32_t {
    if (rt) return (uint32_t)tokb[ibuf * C::M + r];
    return (uint32_t)(itl.row0 + (r < itl.nrows ? r : 0));
  };
  // to tile itl's first stage (its tokens are in LDS): offsets and pointers,
  // and the tokens of the tile after it on their way
  auto bind = [&]() __attribute__((always_inline)) {
    const PnArgPtr q = pn_args();
    const int wi = pn_fresh_s(w);
    const int64_t er = (int64_t)itl.e * N;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int g = wi + 8 * j;
      wb[j] = uni_ptr(q->w_codes + (er + pn_wrow<EPI>(g >> 1, itl.nt, N) + 16 * (g & 1)) * kb2);
    }
    const int64_t wr = er + pn_wrow<EPI>(wi, itl.nt, N);
    wsb = uni_ptr(sfrag ? q->w_sfrag + (wr >> 4) * (K >> 8) * 256 : q->w_scales + wr * kb16);
    pa = uni_ptr(q->a_codes);
    ps = uni_ptr(q->a_scales);
    const int32_t *rt = q->row_token;
#pragma unroll
    for (int j = 0; j < C::NJ; ++j) {
      const int a = wi + 8 * j;
      if (a < 4 * MF)
        oa[j] = src(rt, 16 * a + ri) * (uint32_t)kb2 + pc;
      else if (a < 6 * MF)
        oa[j] = src(rt, 32 * (a - 4 * MF) + (lane >> 1)) * (uint32_t)kb16 + 4u * (uint32_t)(lane & 1);
      else
        oa[j] = 0u;
    }
    phase = 0;
    left = nst;
    if (it + nsl < t_end) {
      nx = pn_locate<MF>(S, it + nsl, ecur, lane);
      tok_dma(nx, ibuf ^ 1);
    }
  };
  // the phase is over: the next one, or the next tile
  auto next_phase = [&]() __attribute__((always_inline)) {
    if (phase == 0 && nmain > nst) {
      const PnArgPtr q = pn_args();
      pa = uni_ptr(q->r_codes);
      ps = uni_ptr(q->r_scales);
      wb[0] = uni_ptr(wb[0] - nst * 64);
      wb[1] = uni_ptr(wb[1] - nst * 64);
      wsb = uni_ptr(wsb - nst * bstep);
      phase = 1;
      left = nst;
    } else if (phase < 2 && nres > 0) {
      phase = 2;
      left = nres;
    } else {
      it += nsl;
      if (it < t_end) {
        itl = nx;
        ibuf ^= 1;
        bind();
      } else {
        phase = 3;
        left = 0x7fffffff;
      }
    }
  };
  // A stage of loads into the slot at LDS address sb, LPS per wave always
  // (placeholders where a stage has none), so that the waits can count.
  // Load j of a stage of codes: 0, 1 weight codes, 2 weight scales, 3 ..
  // activations (codes, then scales).
  auto load = [&](auto j_c, uint32_t sb) __attribute__((always_inline)) {
    constexpr int j = decltype(j_c)::value;
    if constexpr (j < 2) {
      dma16s(wb[j], ob, uni(sb + C::BCODE + (w + 8 * j) * 1024));
    } else if constexpr (j == 2) {
      dma4s(wsb, obs, uni(sb + C::BSCL + w * 256));
    } else if constexpr (j < C::LPS) {
      const int a = w + 8 * (j - 3);
      if (8 * (j - 3) + 7 < 4 * MF || a < 4 * MF)
        dma16s(pa, oa[j - 3], uni(sb + a * 1024));
      else if (8 * (j - 3) + 7 < 6 * MF || a < 6 * MF)
        dma4s(ps, oa[j - 3], uni(sb + C::ASCL + (a - 4 * MF) * 256));
      else
        dma4s(pa, 0u, uni(dummy));
    }
  };
  auto advance = [&]() __attribute__((always_inline)) {
    wb[0] += 64;
    wb[1] += 64;
    wsb += bstep;
    pa += 64;
    ps += 8;
  };
  // the stages that hold no codes: compact residual, or none
  auto issue_rest = [&](uint32_t sb) __attribute__((always_inline)) {
    const PnArgPtr ar = pn_args();
    const uint8_t *any = uni_ptr(ar->a_codes);
    const int wi = pn_fresh_s(w);
#pragma unroll
    for (int j = 0; j < 3; ++j) dma4s(any, 0u, uni(dummy));
    const int t = nres - 1 - left;         // channels 32 t .. 32 t + 31
    const uint8_t *rs = uni_ptr(reinterpret_cast<const uint8_t *>(ar->r_sel) + t * 64);
    // the last stage may hold 16 channels: its upper pieces repeat the lower
    const uint32_t rpc = 32 * t + 16 < ksa ? pc : 16u * (uint32_t)(pcs & 1);
#pragma unroll
    for (int j = 0; j < C::NJ; ++j) {
      const int a = wi + 8 * j;
      if (phase == 2 && a < 4 * MF) {
        const int r = 16 * a + ri;
        const uint32_t row = ar->rsel_rows ? (uint32_t)(itl.row0 + (r < itl.nrows ? r : 0))
                                           : src(ar->row_token, r);
        dma16s(rs, row * (uint32_t)(ksa * 2) + rpc, uni(sb + a * 1024));
      } else {
        dma4s(any, 0u, uni(dummy));
      }
    }
  };
  // starts a stage of loads: true if its LPS loads are load(0) .. (the caller
  // spreads them over its work, then advances), false if they are issued
  auto start = [&](uint32_t sb) __attribute__((always_inline)) -> bool {
    if (left == 0) next_phase();
    --left;
    if (phase < 2) return true;
    issue_rest(sb);
    return false;
  };
  auto loads = [&](uint32_t sb) __attribute__((always_inline)) {
    load(std::integral_constant<int, 0>{}, sb);
    load(std::integral_constant<int, 1>{}, sb);
    load(std::integral_constant<int, 2>{}, sb);
    load(std::integral_constant<int, 3>{}, sb);
    load(std::integral_constant<int, 4>{}, sb);
    load(std::integral_constant<int, 5>{}, sb);
    load(std::integral_constant<int, 6>{}, sb);
    advance();
  };

  if (it < t_end) {
    itl = pn_locate<MF>(S, it, ecur, lane);
    tok_dma(itl, 0);
    wait_vm<0>();
    pn_barrier();
    bind();
    for (int q = 0; q < ns; ++q) {         // ns <= nst: stages of this tile
      --left;
      loads(uni(ring + q * C::SLOT));
    }
    pn_wait<C::LPS>(ns - 1);
    pn_barrier();
  }
  int slot = 0;            // the slot of the stage being multiplied
  PnTile cur = itl;
  while (ct < t_end) {
    const int e = cur.e, nt = cur.nt, row0 = cur.row0, nrows = cur.nrows;
    const float sw = pn_args()->w_gs[2 * e + 1];
    if (cmp && per_expert) {
      for (int i = tid; i < ksa; i += PN_THREADS)
        sel_l[i] = i < p.Ks ? pn_args()->sel[(int64_t)e * p.sel_stride + i] : 0;
      pn_barrier();
    }
    const int nfr = (nrows + 31) >> 5, half = (nfr + 1) >> 1;
    const int fa0 = wm ? half : 0;
    const int mtv = wm ? nfr - half : half;
    const int fb0 = EPI == QD_EPI_SWIGLU ? wn : 2 * wn;
    constexpr int FBS = EPI == QD_EPI_SWIGLU ? 4 : 1;    // the wave's second fragment: fb0 + FBS

    auto run = [&](auto mtv_c) __attribute__((always_inline)) {
      constexpr int MTV = decltype(mtv_c)::value;
      constexpr int MA = MTV > 0 ? MTV : 1;
      f32x16 acc[MA][2];
#pragma unroll
      for (int i = 0; i < MA; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;
      // this lane's operand places in a slot: piece 2 h of its row in
      // fragment fa0 / fb0 (piece 2 h + 1: the address with bit 4 flipped)
      const int r = lane & 31, h = lane >> 5, rr = r & 15;
      const int fo = (r >> 4) * 1024 + rr * 64;
      const int la = fa0 * 2048 + fo + (((2 * h) ^ pn_swz(rr)) << 4);
      const int lb = C::BCODE + fb0 * 2048 + fo + (((2 * h) ^ pn_swz(rr)) << 4);
      const int las = C::ASCL + (32 * fa0 + r) * 8 + 4 * h;
      const int lbs = C::BSCL + (2 * fb0 + (r >> 4)) * 128 + (16 * h + rr) * 4;
      struct AOp {
        uint4 c;
        uint32_t s;
      };
      auto rd_a = [&](const unsigned char *sl, int i, int c) __attribute__((always_inline)) -> AOp {
        AOp o;
        o.c = *reinterpret_cast<const uint4 *>(sl + (c ? la ^ 16 : la) + i * 2048);
        o.s = *reinterpret_cast<const uint32_t *>(sl + las + i * 256);
        return o;
      };
      auto rd_b = [&](const unsigned char *sl, uint4 (&b)[2], int c) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
          b[j] = *reinterpret_cast<const uint4 *>(sl + (c ? lb ^ 16 : lb) + j * FBS * 2048);
      };
      // the barrier of a stage: the next stage has landed, every wave's
      // operands of this one are in registers, so its slot (returned) may be
      // refilled
      auto sync = [&]() __attribute__((always_inline)) -> uint32_t {
        pn_wait<C::LPS>(ns - 2);
        pn_barrier();
        const uint32_t sb = uni(ring + slot * C::SLOT);
        slot = slot + 1 == ns ? 0 : slot + 1;
        return sb;
      };
      auto refill = [&](uint32_t sb) __attribute__((always_inline)) {
        if (start(sb)) loads(sb);
      };
      // RAC: the next selected channel this thread group copies (waves 0..3
      // the even entries of S, 4..7 the odd ones; S is ascending)
      int nk = w >> 2, nsel = 0x7fffffff;
      if (cmp) nsel = nk < p.Ks ? (int)uni((uint32_t)sel_l[nk]) : 0x7fffffff;
      // the selected channels of stage s: decoded weight values into the
      // table (exact: the hardware FP4 conversion with a power-of-two scale
      // and one f16 multiply by the E4M3 scale, as in the operand decode)
      auto copy = [&](const unsigned char *sl, int s) __attribute__((always_inline)) {
        if (nsel >= PN_K * (s + 1)) return;
        const int tb = pn_fresh(tid) & 255, ti = tb & 15;
        const unsigned char *bc = sl + C::BCODE + (tb >> 4) * 1024 + ti * 64;
        const unsigned char *bs = sl + C::BSCL + (tb >> 4) * 128 + ti * 4;
        while (nsel < PN_K * (s + 1)) {     // wave-uniform
          const int el = nsel - PN_K * s;   // >= 0: S is ascending
          const int nk2 = nk + 2;
          const int nxt = nk2 < p.Ks ? sel_l[nk2] : 0x7fffffff;
          const uint32_t byte = bc[(((el >> 5) ^ pn_swz(ti)) << 4) + ((el & 31) >> 1)];
          const uint32_t sbyte = bs[(el >> 6) * 64 + ((el & 63) >> 4)];
          const f16x2 v2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(byte, 256.0f, 0);
          const f16x2 sc = __builtin_bit_cast(f16x2, sbyte << 7);
          *reinterpret_cast<_Float16 *>(lds + L.tab + (tb * ksp + nk) * 2) =
              (el & 1 ? v2[1] : v2[0]) * sc[0];
          nk = nk2;
          nsel = (int)uni((uint32_t)nxt);
        }
      };

      AOp ca;
      uint4 cb[2];
      uint32_t bs[2];
      auto first = [&]() __attribute__((always_inline)) {
        const unsigned char *sl = lds + slot * C::SLOT;
        ca = rd_a(sl, 0, 0);
        rd_b(sl, cb, 0);
#pragma unroll
        for (int j = 0; j < 2; ++j) bs[j] = *reinterpret_cast<const uint32_t *>(sl + lbs + j * FBS * 256);
      };
      if constexpr (MTV > 0) first();
      for (int s = 0; s < nmain; ++s) {
        const unsigned char *sl = lds + slot * C::SLOT;
        if (s == nst) {                    // dense residual: the second pass
#pragma unroll
          for (int i = 0; i < MA; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int q = 0; q < 16; ++q) acc[i][j][q] *= inv_c;
        }
        if (cmp) copy(sl, s);
        if constexpr (MTV == 0) {
          refill(sync());
        } else {
          uint4 nb[2];
          f16x8 bf[4][2];
#pragma unroll
          for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int i = 0; i < MTV; ++i) {
              AOp na;
              const AOp cc = ca;
              const uint4 cbc[2] = {cb[0], cb[1]};
              const uint32_t bsc[2] = {bs[0], bs[1]};
              const bool lastf = i == MTV - 1;
              if (c == 0 && lastf) rd_b(sl, nb, 1);
              if (!lastf) {
                na = rd_a(sl, i + 1, c);
              } else if (c == 0) {
                na = rd_a(sl, 0, 1);
                cb[0] = nb[0];
                cb[1] = nb[1];
              }
              uint32_t sb = 0;
              bool fill = false;
              if (c == 1 && lastf) {
                sb = sync();
                if (s + 1 < nmain) {
                  first();
                  na = ca;
                }
                fill = start(sb);
              }
              const f16x2 ap = scale_pair_of(cc.s, c);
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                if (i == 0) {
#pragma unroll
                  for (int j = 0; j < 2; ++j)
                    bf[q][j] = decode8_sel(word_of(cbc[j], q), scale_pair_of(bsc[j], c), q >= 2);
                }
                const f16x8 af = decode8_sel(word_of(cc.c, q), ap, q >= 2);
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mfma32(af, bf[q][j], acc[i][j]);
                // the refill's loads run under the last fragment's MFMAs
                if (c == 1 && lastf && fill) {
                  switch (q) {
                    case 0: load(std::integral_constant<int, 0>{}, sb);
                            load(std::integral_constant<int, 1>{}, sb); break;
                    case 1: load(std::integral_constant<int, 2>{}, sb);
                            load(std::integral_constant<int, 3>{}, sb); break;
                    case 2: load(std::integral_constant<int, 4>{}, sb);
                            load(std::integral_constant<int, 5>{}, sb); break;
                    default: load(std::integral_constant<int, 6>{}, sb); advance();
                  }
                }
              }
              ca = na;
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
      if (nres > 0) {
        if constexpr (MTV > 0) {
#pragma unroll
          for (int i = 0; i < MA; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int q = 0; q < 16; ++q) acc[i][j][q] *= inv_c;
        }
        for (int t = 0; t < nres; ++t) {
          if constexpr (MTV == 0) {
            refill(sync());
          } else {
            const unsigned char *sl = lds + slot * C::SLOT;
            const bool two = 32 * t + 16 < ksa;
            const int ln = pn_fresh(lane), r = ln & 31, h = ln >> 5, rr = r & 15;
            const int fo = (r >> 4) * 1024 + rr * 64;
            f16x8 ra[2][MA], rb[2][2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              if (c == 0 || two) {
#pragma unroll
                for (int i = 0; i < MTV; ++i)
                  ra[c][i] = *reinterpret_cast<const f16x8 *>(
                      sl + fa0 * 2048 + fo + (((2 * c + h) ^ pn_swz(rr)) << 4) + i * 2048);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                  // table rows are 8-byte aligned: two 8-byte reads
                  const uint2 *q = reinterpret_cast<const uint2 *>(
                      lds + L.tab + ((32 * (fb0 + j * FBS) + r) * ksp + 32 * t + 16 * c + 8 * h) * 2);
                  const uint2 lo = q[0], hi = q[1];
                  rb[c][j] = __builtin_bit_cast(f16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
                }
              }
            }
            refill(sync());
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              if (c == 0 || two) {
#pragma unroll
                for (int i = 0; i < MTV; ++i)
#pragma unroll
                  for (int j = 0; j < 2; ++j) acc[i][j] = mfma32(ra[c][i], rb[c][j], acc[i][j]);
              }
            }
          }
        }
      }
      // ---- epilogue: tensor scales, SwiGLU or plain, bf16 pairs of
      // adjacent columns swapped between neighbouring lanes so that every
      // store writes 4 bytes
      if constexpr (MTV > 0) {
        const float alpha = t_dec * sw;
        const int ln = pn_fresh(lane), h = ln >> 5;
        const bool odd = (ln & 1) != 0;
        const int cpair = (ln & 31) & ~1;
        constexpr int NO = EPI == QD_EPI_SWIGLU ? 1 : 2;
        const int ldo = pn_fresh_s(EPI == QD_EPI_SWIGLU ? (N >> 1) : N);
        unsigned char *obase = reinterpret_cast<unsigned char *>(pn_args()->out);
#pragma unroll
        for (int i = 0; i < MTV; ++i) {
          const int rl = 32 * (fa0 + i) + 4 * h + (odd ? 1 : 0);
          const bool full = 32 * (fa0 + i) + 32 <= nrows;
#pragma unroll
          for (int jj = 0; jj < NO; ++jj) {
            const int cb0 = EPI == QD_EPI_SWIGLU ? nt * 128 + 32 * wn : nt * PN_N + 32 * (fb0 + jj);
            if (cb0 >= ldo) continue;      // the fragment lies past N
            __builtin_amdgcn_sched_barrier(0);   // one fragment's values at a time
            const uint32_t voff = (uint32_t)((row0 + rl) * ldo + cb0 + cpair) * 2u;
            float v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
              if (EPI == QD_EPI_SWIGLU)
                v[q] = swiglu_fast(alpha * acc[i][0][q], alpha * acc[i][1][q]);
              else
                v[q] = alpha * acc[i][jj][q];
            }
#pragma unroll
            for (int q = 0; q < 16; q += 2) {
              const float send = odd ? v[q] : v[q + 1];
              const float x = __int_as_float(
                  __builtin_amdgcn_mov_dpp(__float_as_int(send), 0xB1, 0xF, 0xF, false));
              const f32x2_t pr = odd ? f32x2_t{x, v[q + 1]} : f32x2_t{v[q], x};
              const uint32_t pk = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2_t));
              const int qr = 8 * (q >> 2) + (q & 3);
              if (full || rl + qr < nrows) {
                *reinterpret_cast<uint32_t *>(obase + (size_t)(qr * ldo * 2) + voff) = pk;
                vmax = fmaxf(vmax, fmaxf(fabsf(__uint_as_float(pk << 16)),
                                         fabsf(__uint_as_float(pk & 0xFFFF0000u))));
              }
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
  }
  wait_vm<0>();
  const float m = block_max(vmax, red);
  qdg::put_amax(p, m);
}

template <int MF, int EPI>
void launch_panel_epi(const GemmArgs &p, const PnDeal &deal, int grid, int ns, int dense, int lds,
                      hipStream_t s) {
  auto kern = gemm_panel_kernel<MF, EPI>;
  static const bool attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               PN_LDS_MAX) == hipSuccess;
  (void)attr;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(PN_THREADS), (size_t)lds, s, p, deal, ns,
                     dense);
}

// one compiled tile height each (gemm_panel_<MF>.hip)
template <int MF>
void launch_panel(const GemmArgs &p, int epi, const PnDeal &deal, int grid, int ns, int dense,
                  int lds, hipStream_t s);

}  // namespace qdp
