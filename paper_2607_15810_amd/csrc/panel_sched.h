// The tile schedule of the persistent prefill GEMMs (tiles of up to 64 MF rows
// of one expert x 256 weight rows, one workgroup of eight waves per CU), and
// the waits of their LDS rings.
#pragma once
#include <algorithm>
#include <cmath>

#include "common.h"
#include "lds_dma.h"
#include "tile_sched.h"

namespace qdp {

using namespace qd;
using namespace qdl;

constexpr int PN_THREADS = 512;
constexpr int PN_N = 256;
constexpr int PN_EMAX = 1024;
constexpr int PN_NSMAX = 6;
constexpr int PN_LDS_MAX = 160 * 1024 - 512;   // dynamic LDS beside the static arrays
constexpr int PN_LDS_2WG = 80 * 1024 - 512;    // the same for two workgroups per CU

template <int LPS>
__device__ __forceinline__ void pn_wait(int stages) {
  switch (stages) {      // uniform
    case 0: wait_vm<0>(); break;
    case 1: wait_vm<LPS>(); break;
    case 2: wait_vm<2 * LPS>(); break;
    case 3: wait_vm<3 * LPS>(); break;
    default: wait_vm<4 * LPS>(); break;
  }
}
// this wave's LDS reads and writes are done, then the workgroup's barrier
__device__ __forceinline__ void pn_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// the same value, computed anew from here on: keeps the address arithmetic of
// the parts outside the K loop from being hoisted above it, where it would
// hold registers the accumulators need
__device__ __forceinline__ int pn_fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ int pn_fresh_s(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

struct PnTile {
  int e, row0, nrows, nt;
};

// An expert's nf 32-row fragments in n tiles of equal height to one fragment,
// q = nf / n: the first fragment of tile i (nf for i = n).  No product of two
// large counts: one expert may hold 2^19 fragments and more.
__host__ __device__ inline int pn_cut(int nf, int n, int q, int i) {
  const int r = nf - q * n;
  return i * q + (i < r ? i : r);
}

// How the tiles are dealt to the XCDs: units of cg M-tiles x nb weight-row
// tiles; an M-tile's ntn weight-row tiles make nsp = ntn / nb units (nsp > 1
// only with cg = 1).  XCD x walks its units x, x + 8, .., the weight-row tiles
// of an M-tile innermost.
struct PnDeal {
  int cg, nb, nsp;
};
struct PnPlace {
  int mt, nt;
};
// (Integer divisions run on the vector unit: their results are made scalar.)
__host__ __device__ inline int pn_div(int a, int b) {
#ifdef __HIP_DEVICE_COMPILE__
  return (int)uni((uint32_t)a / (uint32_t)b);
#else
  return a / b;
#endif
}
// the tile at place l of XCD xcd's walk
__host__ __device__ inline PnPlace pn_place(const PnDeal &d, int xcd, int l) {
  const int gt = d.cg * d.nb;
  const int q = pn_div(l, gt), rem = l - q * gt;
  const int j = pn_div(rem, d.nb), u = xcd + 8 * q;
  const int g = d.nsp == 1 ? u : pn_div(u, d.nsp);
  return {g * d.cg + j, (u - g * d.nsp) * d.nb + rem - j * d.nb};
}
// the length of that walk over mts M-tiles
__host__ __device__ inline int pn_length(const PnDeal &d, int xcd, int mts) {
  const int ng = pn_div(mts + d.cg - 1, d.cg), nu = ng * d.nsp;
  const int nq = nu > xcd ? (nu - xcd + 7) >> 3 : 0;
  const bool last = nu > 0 && ((nu - 1) & 7) == xcd;       // the group that may be short
  return (nq * d.cg - (last ? ng * d.cg - mts : 0)) * d.nb;
}

// The M-tiles run over the experts in the order of perm (mpre: M-tiles before
// each place of it); workgroup b takes every (G / 8)-th tile, from b / 8 on, of
// the walk of XCD b % 8.  Places of the walk are visited in increasing order, so
// the cursor into perm advances by a wave ballot over the next 64 places.
struct PnSched {
  const int32_t *offs, *mpre;
  const uint16_t *perm;
  int E;
  PnDeal d;
  int xcd;
};

template <int MF>
__device__ __forceinline__ PnTile pn_locate(const PnSched &S, int l, int &cur, int lane) {
  const PnPlace pl = pn_place(S.d, S.xcd, l);
  const int mt = pl.mt;
  for (;;) {
    const int c = cur + 1 + lane;
    const bool le = c <= S.E && S.mpre[c] <= mt;
    const int adv = __popcll(__ballot(le));
    cur = (int)uni((uint32_t)(cur + adv));
    if (adv < 64) break;
  }
  PnTile tl;
  tl.e = (int)uni((uint32_t)S.perm[cur]);
  const int o0 = (int)uni((uint32_t)S.offs[tl.e]);
  const int rows = (int)uni((uint32_t)S.offs[tl.e + 1]) - o0;
  const int i = mt - (int)uni((uint32_t)S.mpre[cur]);
  const int nf = (rows + 31) >> 5, n = (nf + 2 * MF - 1) / (2 * MF);
  const int h = (int)uni((uint32_t)nf / (uint32_t)n);
  const int f0 = pn_cut(nf, n, h, i), f1 = pn_cut(nf, n, h, i + 1);
  tl.row0 = o0 + 32 * f0;
  tl.nrows = min(32 * f1, rows) - 32 * f0;
  tl.nt = pl.nt;
  return tl;
}

// tiles of the walk of S's XCD
__device__ __forceinline__ int pn_walk(const PnSched &S) {
  return pn_length(S.d, S.xcd, (int)uni((uint32_t)S.mpre[S.E]));
}

// The schedule (two experts per thread, E <= 1024): row offsets, the experts
// sorted by the height of their tiles, tallest first (then by index), and the
// M-tiles before each.  The caller's barrier makes mpre visible.
template <int MF>
__device__ __forceinline__ void pn_schedule(const int32_t *offsets, int64_t rows, int E,
                                            int32_t *offs, int32_t *mpre, uint16_t *perm,
                                            int *sh_w, int (*sh_c)[2 * MF + 1]) {
  const int tid = threadIdx.x, lane = tid & 63, w = (int)uni((uint32_t)tid >> 6);
  int cnt[2], cls[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = 2 * tid + q;
    int o0 = 0, o1 = 0;
    if (e <= E) {
      o0 = offsets ? offsets[e] : (e == 0 ? 0 : (int)rows);
      offs[e] = o0;
    }
    if (e < E) o1 = offsets ? offsets[e + 1] : (int)rows;
    const int nf = e < E ? (max(o1 - o0, 0) + 31) / 32 : 0;
    cnt[q] = (nf + 2 * MF - 1) / (2 * MF);
    // sorting class: 2 MF - height of the expert's tallest tile (2 MF: none)
    cls[q] = e >= E ? -1 : nf == 0 ? 2 * MF : 2 * MF - (nf + cnt[q] - 1) / cnt[q];
  }
  if (E == PN_EMAX && tid == 0) offs[E] = offsets ? offsets[E] : (int)rows;
  int pos[2] = {0, 0};
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int c = 0; c <= 2 * MF; ++c) {
    const uint64_t b0 = __ballot(cls[0] == c), b1 = __ballot(cls[1] == c);
    const int below = __popcll(b0 & lt) + __popcll(b1 & lt);
    if (cls[0] == c) pos[0] = below;
    if (cls[1] == c) pos[1] = below + (cls[0] == c ? 1 : 0);
    if (lane == 0) sh_c[w][c] = __popcll(b0) + __popcll(b1);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (cls[q] < 0) continue;
    int at = pos[q];
    for (int c = 0; c < cls[q]; ++c)
      for (int ww = 0; ww < 8; ++ww) at += sh_c[ww][c];
    for (int ww = 0; ww < w; ++ww) at += sh_c[ww][cls[q]];
    perm[at] = (uint16_t)(2 * tid + q);
    mpre[at] = cnt[q];
  }
  __syncthreads();
  // M-tile counts to prefix sums, in place
  int tsum = 0;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    cnt[q] = 2 * tid + q < E ? mpre[2 * tid + q] : 0;
    tsum += cnt[q];
  }
  int xs = tsum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(xs, o, 64);
    if (lane >= o) xs += y;
  }
  if (lane == 63) sh_w[w] = xs;
  __syncthreads();
  int base = xs - tsum;
  for (int ww = 0; ww < w; ++ww) base += sh_w[ww];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = 2 * tid + q;
    if (e <= E) mpre[e] = base;
    base += cnt[q];
  }
  if (E == PN_EMAX && tid == PN_THREADS - 1) mpre[E] = base;
}

// Expected experts with more than x rows, of one with a normal count (E = 1: its
// rows are known), and rounds of the 256 CUs that mts expected M-tiles of ntn
// tiles each take: what mts has past a whole number is the chance of one more.
inline double pn_above(double x, double mean, double sd, int E) {
  if (E == 1) return mean > x ? 1.0 : 0.0;
  return 0.5 * erfc((x - mean) / (sd * 1.4142135623730951));
}
inline double pn_rounds(double mts, int ntn) {
  const double whole = std::floor(mts + 0.02), more = 1.0 - std::exp(std::min(0.0, whole - mts));
  const auto rounds = [&](double m) { return std::max(1.0, std::ceil(m * ntn / 256.0)); };
  return rounds(whole) * (1.0 - more) + rounds(whole + 1.0) * more;
}

// The same where the M-tiles vary by sd about mts: few experts of a count near a
// whole number of tiles may all need one more.
inline double pn_rounds(double mts, double sd, int ntn) {
  const auto rounds = [&](double m) { return std::max(1.0, std::ceil(m * ntn / 256.0)); };
  if (sd < 0.15) return rounds(std::floor(mts + 0.5));
  if (sd > 20.0) return rounds(mts);
  const double last = std::ceil(mts + 3.0 * sd);
  double t = 0.0, below = 0.0;
  for (double m = std::max(1.0, std::floor(mts - 3.0 * sd)); m <= last; m += 1.0) {
    const double upto = m < last ? 0.5 * erfc((mts - m - 0.5) / (sd * 1.4142135623730951)) : 1.0;
    t += (upto - below) * rounds(m);
    below = upto;
  }
  return t;
}

// Expected tiles of `tall` rows that an expert has with more than `cut` rows in
// them (cut 0: all of its tiles): those that all but the rarest experts fill, then
// the tail.  *var: the variance of their number.
inline double pn_tiles(double mean, double sd, int E, double tall, double cut,
                       double *var = nullptr) {
  const double j0 = std::max(0.0, std::floor((mean - 8.0 * sd) / tall));
  double n = j0, v = 0.0;
  for (double j = j0; tall * j <= mean + 8.0 * sd; j += 1.0) {
    const double p = pn_above(tall * j + cut, mean, sd, E);
    n += p;
    v += p * (1.0 - p);
  }
  if (var) *var = v;
  return n;
}

// The tile height with the least estimated time: whole rounds of the 256 CUs,
// each the time of a tile of average height.  The expected number of tiles is
// that of uniform routing (normal counts per expert).  One tile more may begin a
// round (100 +- 10 rows on each of 64 experts, 2048 weight rows: 128-row tiles make
// 512 tiles of them, two rounds, in six of seven draws, and a third round for eight
// in the other: 125 us against 104 with 192-row tiles).  64-row tiles on two
// workgroups per CU (two64: they fit) take 0.74 of the time once there is more than a
// round of them, as long as they hold an average expert (56 rows on each of 128
// experts, K = 4096, 768 weight rows: 86 us against 109 with the wide kernel; 80 rows,
// K = 2048 twice: 120 against 111 with the tile kernel).
// fixed: a tile's fixed time, in that of a 32-row fragment; spread: rounds with the
// spread of the tiles' number.
// ns_of(mf): the ring depth that height leaves room for (< 2: none).
struct PnHeight {
  int mf, ns, cg;
  double mts;              // M-tiles expected
  double time;             // in that of a 32-row fragment of a tile
};
constexpr double PN_TWO = 0.74;
template <typename F>
inline PnHeight pn_height(int64_t rows, int E, int ntn, double fixed, bool spread, bool two64,
                          F ns_of) {
  PnHeight h{};
  const double mean = (double)rows / E, sd = std::max(0.5, sqrt(mean));
  double best = 0.0;
  for (const int mf : {1, 2, 3, 5}) {
    const int ns = ns_of(mf);
    if (ns < 2) continue;
    double var;
    const double n = std::max(pn_tiles(mean, sd, E, 64.0 * mf, 0.0, &var), 1.0 / E);
    const double r = spread ? pn_rounds(n * E, sqrt(var * E), ntn) : pn_rounds(n * E, ntn);
    double t = r * (fixed + (mean / 32.0 + 0.5) / n);
    if (mf == 1 && two64 && n * E * ntn > 256.0 && mean <= 64.0) t *= PN_TWO;
    if (h.mf == 0 || t < 0.995 * best) {     // even: the lower, its ring is deeper
      best = t;
      // M-tiles dealt to the XCDs in the number an average expert has
      h = {mf, ns, std::max(1, (int)std::min(8.0, n + 0.5)), n * E, t};
    }
  }
  return h;
}

// Prices of the W4A4 kernels' tiles, in the time of one 32-row fragment through
// one 128-element stage of K; nst: those stages (of both passes with the dense
// residual).  Fitted to 706 GEMMs (1 to 128 experts of 4 to 3000 rows, K 384 to
// 4096, N 768 to 8192, no residual, K_s = K / 32 and K / 2, each on every kernel and
// tile height): the choice is 0.7% above the fastest on average, 14% at worst.
// The panel kernel's fixed part is the decode of its weights and barriers of every
// stage, and once per tile its start and epilogue.
inline double panel_fixed(double nst) { return 4.4 + 6.0 / nst; }

// The tile kernel: 256 x 128 tiles, each cut at 256 rows and priced by its fullest
// 32, 64, 128 or 256, on 512 workgroups at a time.  A round of at most half of
// them runs one per CU, the faster for it.
inline double tile_time(int64_t rows, int E, int ntn, double nst) {
  const double mean = (double)rows / E, sd = std::max(0.5, sqrt(mean));
  const auto with = [&](double cut) { return pn_tiles(mean, sd, E, 256.0, cut); };
  const double n = std::max(with(0.0), 1.0 / E);
  const double price = (5.6 * n + 1.4 * with(32.0) + 1.3 * with(64.0) + 3.7 * with(128.0)) / n;
  const auto rounds = [&](double mts) {
    const double x = std::max(mts, 1.0) * ntn / 512.0, whole = std::floor(x), r = x - whole;
    return whole + (r <= 0.0 ? 0.0 : r > 0.5 ? 1.0 : whole > 0.0 ? 0.6 : 0.68);
  };
  const double mts = n * E, whole = std::floor(mts + 0.02);
  const double more = 1.0 - std::exp(std::min(0.0, whole - mts));
  return (rounds(whole) * (1.0 - more) + rounds(whole + 1.0) * more) * (price + 1.8 / nst);
}
// rounds of its workgroups
inline double tile_rounds(int64_t rows, int E, int ntn) {
  const double mean = (double)rows / E, sd = std::max(0.5, sqrt(mean));
  return pn_tiles(mean, sd, E, 256.0, 0.0) * E * ntn / 512.0;
}

// The deal of h's M-tiles over a grid of workgroups.  Whole M-tiles, as many
// together as an average expert has, share most in an XCD's L2, and from 64 such
// units on they load the XCDs evenly.  With fewer the largest units are taken
// that need no more rounds of an XCD's workgroups than single tiles would: one
// M-tile, or one expert's eight, would otherwise keep seven XCDs idle.
inline PnDeal pn_deal(const PnHeight &h, int ntn, int grid) {
  if (h.mts >= 64.0 * h.cg) return {h.cg, ntn, 1};
  const int m = std::max(1, (int)std::ceil(h.mts - 0.2)), wgs = grid / 8;
  const auto rounds = [&](int cg, int nb) {
    const int units = (m + cg - 1) / cg * (ntn / nb);
    return ((units + 7) / 8 * cg * nb + wgs - 1) / wgs;
  };
  const int least = rounds(1, 1);
  if (rounds(h.cg, ntn) <= least) return {h.cg, ntn, 1};
  int nb = ntn;
  while (nb > 1 && (ntn % nb != 0 || rounds(1, nb) > least)) --nb;
  return {1, nb, ntn / nb};
}

}  // namespace qdp
