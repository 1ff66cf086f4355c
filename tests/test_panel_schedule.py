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
extern "C" void cuts(int nf, int n, int *out) {
  for (int i = 0; i <= n; ++i) out[i] = qdp::pn_cut(nf, n, nf / n, i);
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
    return ctypes.CDLL(so)


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
