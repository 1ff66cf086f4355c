"""GPU parity of the grouped GEMM's kernel for a handful of rows: one row,
more than the 8 rows of a pass on one expert, empty experts, more experts than
one scan of the offsets holds, K split over one, two and four waves, K with a
part of a 256-element chunk, and the residual listed from its bitmap (one
token through the layer)."""

import zlib

import numpy as np
import pytest
import torch

from oracle import layer as OL, rac as OR
from paper_2607_15810_amd import ops, synth
from paper_2607_15810_amd import quads as Q

from helpers import check_close_bf16, np_bf16, oracle_bank

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q.lib()
    yield


CASES = [
    # name, experts, {expert: rows}, K, N, Ks
    ("one_row", 1, {0: 1}, 256, 32, 4),
    ("passes", 3, {0: 8, 1: 9, 2: 17}, 512, 96, 16),
    ("k64", 2, {0: 2, 1: 1}, 64, 64, 0),
    ("k320", 4, {1: 3, 3: 7}, 320, 128, 24),
    ("k1088_four_waves", 2, {0: 5, 1: 2}, 1088, 64, 32),
    ("many_experts", 300, {0: 1, 127: 2, 128: 1, 299: 3}, 512, 64, 8),
    ("second_round", 40, {e: 2 for e in range(40)}, 256, 2048, 8),
]


@pytest.mark.parametrize("epi", [Q.QD_EPI_NONE, Q.QD_EPI_SWIGLU], ids=["plain", "swiglu"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_few_rows_gemm(case, epi):
    name, E, per, K, N, Ks = case
    counts = np.zeros(E, np.int64)
    for e, n in per.items():
        counts[e] = n
    live = np.nonzero(counts)[0]
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offsets[-1])
    T = max(1, R // 2)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    g = torch.Generator().manual_seed(zlib.crc32(name.encode()))
    x = torch.randn((T, K), generator=g)
    x[:, ::13] *= 20.0
    x = x.to(torch.bfloat16)
    wb = torch.zeros((E, N, K), dtype=torch.bfloat16)
    for e in live:
        wb[e] = (torch.randn((N, K), generator=g) * 0.02).to(torch.bfloat16)
    tok = rng.integers(0, T, R).astype(np.int32)
    w, W = ops.quantize_weight(wb.to(DEV)), oracle_bank(wb, live)
    xg = x.to(DEV)
    xq, scores, ramax = ops.quantize_act(xg, rac=True)
    act = OR.rac_activation(np_bf16(x), Ks)
    sel = rq = None
    if Ks:
        sel, rq, _, _ = ops.select_channels(xg, xq, Ks, scores, ramax)
    out, amax = ops.grouped_gemm(xq, w, R, torch.from_numpy(tok).to(DEV),
                                 torch.from_numpy(offsets).to(DEV) if E > 1 else None, rq, sel,
                                 epi, want_amax=True)
    gu, mag = OL.w13_stage(act["xq"], act["rq"] if Ks else None, tok, offsets, W)
    ref = gu
    if epi == Q.QD_EPI_SWIGLU:
        I = N // 2
        ref = OL.silu(gu[:, :I]) * gu[:, I:]
        mag = (np.abs(OL.silu(gu[:, :I])) * mag[:, I:] + 1.1 * np.abs(gu[:, I:]) * mag[:, :I])
    check_close_bf16(np_bf16(out), ref, mag, name)
    assert amax.max().item() == np.max(np.abs(np_bf16(out)))


@pytest.mark.parametrize("T,H,I,Ks", [(1, 512, 128, 8), (3, 256, 192, 256), (2, 4096, 64, 128)])
def test_few_tokens_layer(T, H, I, Ks):
    """The layer on one to three tokens: the selection reaches the W13 kernel
    as a bitmap, and the kernel lists it."""
    E, k = 16, 4
    inp = synth.small_moe("few", T, H, E, k, I, Ks, seed=3)
    w13, w2 = ops.quantize_weight(inp.w13.to(DEV)), ops.quantize_weight(inp.w2.to(DEV))
    lay = ops.MoELayer(w13, w2, T, k, Ks)
    y = lay(inp.x.to(DEV), inp.logits.to(DEV))
    torch.cuda.synchronize()
    ref = OL.moe_layer(inp.x.float().numpy(), inp.logits.numpy(), oracle_bank(inp.w13),
                       oracle_bank(inp.w2), k, Ks)
    v = lay.views()
    assert np.array_equal(v["sel"].cpu().numpy(), ref["act"]["sel"])
    rel = np.linalg.norm(np_bf16(y) - ref["yb"]) / np.linalg.norm(ref["yb"])
    assert rel <= 1e-3, f"free-running rel-L2 {rel:.3e}"
