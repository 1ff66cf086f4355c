"""The weight quantiser at the edges of its work split (256 blocks of 16
elements per workgroup and pass): sizes with and without a fragment-ordered
copy of the scales, ragged last passes, groups with many passes per workgroup.
Codes, scales and tensor scales are those of the oracle, bit for bit; the
fragment-ordered copy is the one the packing call makes of them."""

import numpy as np
import pytest
import torch

from oracle import quant as OQ
from paper_2607_15810_amd import ops
from paper_2607_15810_amd import quads as Q

from helpers import assert_nvfp4_equal

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q.lib()
    yield


@pytest.mark.parametrize("shape", [(1, 1, 16), (3, 7, 48), (2, 255, 16), (2, 257, 16), (2, 33, 272),
                                   (3, 16, 256), (2, 48, 768), (2, 1040, 1024), (1, 4112, 1280)])
def test_quantize_weight_edges(shape):
    G, R, C = shape
    rng = np.random.default_rng(R * 31 + C)
    w = torch.from_numpy(rng.standard_normal(shape) * 0.05).to(torch.bfloat16)
    w[:, R // 2] = 0.0                      # zero blocks
    w[G - 1, R - 1, C - 1] = 7.0            # the amax in the last block
    q = ops.quantize_weight(w.to(DEV))
    for g in range(G):
        ref = OQ.quantize(w[g].float().numpy())
        one = ops.NVFP4Tensor(q.codes[g:g + 1], q.scales[g:g + 1], q.gscale[g:g + 1], 1, R, C)
        assert_nvfp4_equal(one, ref, f"group {g}")
    has = R % 16 == 0 and C % 256 == 0
    assert (q.scales_frag is not None) == has
    if has:
        assert torch.equal(q.scales_frag, ops.pack_frag_scales(q))
