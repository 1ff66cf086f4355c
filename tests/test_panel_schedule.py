"""The persistent prefill GEMMs' tile schedule on the host: panel_sched.h's own
integer arithmetic, compiled for the CPU."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_15810_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include "panel_sched.h"
#include "gemm_wide.h"
extern "C" void cuts(int nf, int n, int *out) {
  for (int i = 0; i <= n; ++i) out[i] = qdp::pn_cut(nf, n, nf / n, i);
}
extern "C" void walk(int cg, int nb, int nsp, int mts, int *len, int *seen) {
  const qdp::PnDeal d{cg, nb, nsp};
  for (int x = 0; x < 8; ++x) {
    len[x] = qdp::pn_length(d, x, mts);
    for (int l = 0; l < len[x]; ++l) {
      const qdp::PnPlace p = qdp::pn_place(d, x, l);
      if (p.mt < 0 || p.mt >= mts || p.nt < 0 || p.nt >= nb * nsp) { seen[0] = -1; return; }
      ++seen[p.mt * nb * nsp + p.nt];
    }
  }
}
extern "C" void height(long rows, int E, int ntn, double nst, int two64, int *out) {
  const qdp::PnHeight h =
      qdp::pn_height(rows, E, ntn, qdp::panel_fixed(nst), false, two64 != 0,
                     [](int) { return 4; });
  out[0] = h.mf; out[1] = h.cg; out[2] = (int)h.mts;
}
// times of the panel kernel, of the tile kernel (no residual) and of the wide one
extern "C" void times(long rows, int E, int ntn, double nst, double *out) {
  out[0] = qdp::pn_height(rows, E, ntn, qdp::panel_fixed(nst), false, true,
                          [](int) { return 4; }).time;
  out[1] = qdp::tile_time(rows, E, 2 * ntn, nst);
  out[2] = qdw::wide_time(rows, E, ntn, nst);
}
extern "C" int spread_height(long rows, int E, int ntn, double fixed) {
  return qdp::pn_height(rows, E, ntn, fixed, true, false, [](int) { return 4; }).mf;
}
extern "C" double spread_rounds(double mts, double sd, int ntn) {
  return qdp::pn_rounds(mts, sd, ntn);
}
extern "C" void deal(double mts, int cg, int ntn, int grid, int *out) {
  const qdp::PnDeal d = qdp::pn_deal(qdp::PnHeight{1, 2, cg, mts, 0.0}, ntn, grid);
  out[0] = d.cg; out[1] = d.nb; out[2] = d.nsp;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("sched")
    src, so = str(d / "sched.hip"), str(d / "sched.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17",
                        "-fPIC", "-shared", "-I", CSRC, src, "-o", so],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = ctypes.CDLL(so)
    lib.spread_rounds.restype = ctypes.c_double
    return lib


@pytest.mark.parametrize("mf", [1, 2, 3, 5])
@pytest.mark.parametrize("rows", [1, 31, 33, 320, 321, 641, 5000, 6_000_000, 8_388_608,
                                  16_777_215])
def test_tiles_cover_an_expert(host, rows, mf):
    """An expert's tiles follow one another from its first fragment to its
    last, none taller than 2 MF fragments, none more than one fragment taller
    than another."""
    nf = (rows + 31) // 32
    n = -(-nf // (2 * mf))
    out = np.empty(n + 1, np.int32)
    host.cuts(nf, n, out.ctypes.data_as(ctypes.c_void_p))
    h = np.diff(out)
    assert out[0] == 0 and out[-1] == nf
    assert h.min() >= 1 and h.max() <= 2 * mf and h.max() - h.min() <= 1


def _ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


@pytest.mark.parametrize("ntn", [1, 2, 3, 6, 12, 16, 35])
def test_deal_covers_every_tile_evenly(host, ntn):
    """Each tile is walked once, whatever the units; with few M-tiles no XCD
    needs more rounds of its workgroups than an even deal would."""
    for mts in list(range(1, 40)) + [63, 64, 65, 131, 512]:
        for cg in (1, 2, 3, 8):
            grid = min(256, -(-(mts + 1) * ntn // 8) * 8)
            d = np.empty(3, np.int32)
            host.deal(ctypes.c_double(mts), cg, ntn, grid, _ptr(d))
            c, nb, nsp = (int(v) for v in d)
            assert nb * nsp == ntn and (c == 1 or nsp == 1) and c in (1, cg)
            for real in (mts + 5, mts):          # the routing may make more than expected
                length, seen = np.zeros(8, np.int32), np.zeros((real, ntn), np.int32)
                host.walk(c, nb, nsp, real, _ptr(length), _ptr(seen))
                assert np.all(seen == 1), (real, cg, ntn)
            if mts < 64 * cg:
                assert -(-length.max() // (grid // 8)) <= -(-mts * ntn // grid), (mts, cg, ntn)
            else:
                assert (c, nb) == (cg, ntn)


@pytest.mark.parametrize("rows,E,ntn,nst,two64,mf", [
    (128 * 56, 128, 3, 32, True, 1),       # two workgroups per CU on more than a round
    (128 * 90, 128, 3, 32, True, 2),       # more than one such tile per expert: taller ones
    (128 * 90, 128, 3, 32, False, 2),
    (128 * 49, 128, 12, 32, True, 1),
    (64 * 100, 64, 8, 16, False, 3),       # 512 tiles of 128 rows, if no expert has more
    (128 * 145, 128, 3, 16, False, 3),     # two rounds, where 128-row tiles make three
    (128 * 512, 128, 6, 16, True, 5),
    (1, 1, 1, 16, True, 1),
])
def test_tile_height(host, rows, E, ntn, nst, two64, mf):
    out = np.empty(3, np.int32)
    host.height(ctypes.c_long(rows), E, ntn, ctypes.c_double(nst), int(two64), _ptr(out))
    assert out[0] == mf


def test_tile_height_expects_the_tiles(host):
    """The expected M-tiles at large counts per expert, in a bounded number of
    steps."""
    out = np.empty(3, np.int32)
    for rows, E in ((1 << 24, 1), (1 << 24, 2), (1 << 22, 128)):
        host.height(ctypes.c_long(rows), E, 1, ctypes.c_double(16), 0, _ptr(out))
        least = rows / (64 * out[0])
        assert least <= out[2] + 1 and out[2] <= least + E


@pytest.mark.parametrize("rows,E,ntn,nst,fastest", [
    # measured fastest by 4% or more (us: panel, tile, wide kernel)
    (128 * 80, 128, 12, 32, 2),        # 403, 412, 371
    (64 * 80, 64, 3, 16, 2),           # 42, 38, 35
    (64 * 80, 64, 12, 32, 2),          # 206, 210, 191
    (128 * 125, 128, 6, 16, 0),
    (128 * 512, 128, 6, 16, 0),        # half of the experts need a third tile of 256
    (32 * 30, 32, 8, 5, 1),            # 16.0, 13.3
    (16 * 80, 16, 8, 7, 1),            # a few tiles: twice as many of half the width
    (256, 1, 4, 16, 0),                # an idle chip: lower tiles, more of them
    (1024 * 200, 1024, 1, 8, 2),
])
def test_fastest_kernel_by_estimate(host, rows, E, ntn, nst, fastest):
    t = np.empty(3)
    host.times(ctypes.c_long(rows), E, ntn, ctypes.c_double(nst), _ptr(t))
    if nst % 2:
        t[2] = np.inf                  # the wide kernel takes whole 256-element stages
    assert int(np.argmin(t)) == fastest, t


# test_gpu_rows.py's calls of each height: rows per expert on 128 experts, N = 1536
ROWS_HEIGHTS = [(30, 1), (88, 2), (145, 3), (250, 5)]


@pytest.mark.parametrize("fixed", [2.0, 7.0], ids=["fp8", "w4a16"])
@pytest.mark.parametrize("mean,mf", ROWS_HEIGHTS)
def test_rows_height(host, mean, mf, fixed):
    for rows in (128 * mean - 60, 128 * mean + 60):
        assert host.spread_height(ctypes.c_long(rows), 128, 6, ctypes.c_double(fixed)) == mf


@pytest.mark.parametrize("rows,E,ntn,fixed,mf", [
    (8 * 264, 8, 12, 2.0, 3),          # 128-row tiles: 192 to 288 of them for 256 CUs
    (64 * 260, 64, 3, 2.0, 5),
    (128 * 512, 128, 6, 2.0, 5),
    (128 * 4, 128, 6, 7.0, 1),
])
def test_rows_height_with_the_spread(host, rows, E, ntn, fixed, mf):
    assert host.spread_height(ctypes.c_long(rows), E, ntn, ctypes.c_double(fixed)) == mf


def test_rounds_with_the_spread(host):
    """The expected rounds of a normal number of M-tiles, by sampling."""
    rng = np.random.default_rng(3)
    for mts, sd, ntn in ((20.0, 1.4, 12), (85.0, 3.0, 3), (40.3, 0.5, 6), (128.0, 0.0, 6)):
        m = np.maximum(np.rint(mts + sd * rng.standard_normal(200_000)), 1)
        ref = np.maximum(np.ceil(m * ntn / 256), 1).mean()
        got = host.spread_rounds(ctypes.c_double(mts), ctypes.c_double(sd), ntn)
        assert abs(got - ref) < 0.02, (mts, sd, ntn, got, ref)
