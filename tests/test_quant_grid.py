"""The workgroups of the activation quantiser, from quant_dev.h's own host code."""

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
#include "quant_dev.h"
extern "C" int grid(long rows, long cols, int rac, int *out) {
  qdq::quant_grid(rows, cols, rac != 0, out[0], out[1]);
  return qdq::kScoreMaxRows;
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("grid")
    src, so = str(d / "grid.hip"), str(d / "grid.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17",
                        "-fPIC", "-shared", "-I", CSRC, src, "-o", so],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(so)


@pytest.mark.parametrize("rows,cols,least,most", [
    (64, 2048, 32, 32),                # one row block each
    (2000, 2048, 200, 256),            # few rows: the atomics at the end count
    (8192, 2048, 400, 512),
    (8192, 4096, 900, 1024),           # many: the waves in flight do
    (32768, 4096, 900, 1024),
    (2 ** 24, 256, 1, 1024),
])
def test_rac_grid(host, rows, cols, least, most):
    out = np.zeros(2, np.int32)
    bound = host.grid(ctypes.c_long(rows), ctypes.c_long(cols), 1,
                      out.ctypes.data_as(ctypes.c_void_p))
    gx, gy = (int(v) for v in out)
    assert 256 * gx >= cols and least <= gx * gy <= most
    assert -(-rows // (16 * gy)) <= bound      # the exact score sums' terms per thread
