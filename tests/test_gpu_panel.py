"""GPU parity of the grouped GEMM's panel, tile and wide kernels at the edges of
their tiles: row counts around its 32-row fragments and around each tile height (64, 128,
192, 256, 320 rows), widths that are no multiple of 256 weight rows, K of two
and three stages (three: no fragment-ordered scales), every form of the
residual, and the largest expert count of its schedule.

Against the oracle's float64 contraction of its own quantised operands, with
the tolerance every GEMM stage has."""

import zlib

import numpy as np
import pytest
import torch

from oracle import layer as OL, rac as OR
from paper_2607_15810_amd import ops
from paper_2607_15810_amd import quads as Q

from helpers import assert_nvfp4_equal, check_close_bf16, np_bf16, oracle_bank

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q.lib()
    yield


CASES = [
    # name, rows per expert, K, N, Ks, gathered rows
    ("few_rows_k384", [1, 31, 32, 33, 0, 5], 384, 256, 16, True),
    ("k384_half_tile", [63, 64, 65, 0], 384, 128, 0, False),
    ("k256_two_stages", [70, 64, 65, 96], 256, 384, 24, True),
    ("around_128", [127, 128, 129, 97], 512, 256, 40, True),
    ("around_192", [191, 192, 193, 129], 512, 384, 8, True),
    ("around_320", [319, 320, 321, 289], 512, 256, 16, True),
    ("two_tiles", [640, 641, 1, 330], 256, 128, 32, False),
    ("one_expert", [333], 768, 256, 48, False),
    ("dense_residual", [150, 60, 100], 384, 256, 200, True),
    ("dense_residual_320", [300, 321], 512, 128, 160, False),
    ("largest_table", [90, 70], 256, 256, 144, True),
    # 64-row tiles on two workgroups per CU, 600 of them for 512: without
    # and with the dense residual, and beside a table at K of two stages
    ("two_per_cu", [9, 33, 0, 64, 65, 1, 31, 32] * 25, 384, 768, 0, False),
    ("two_per_cu_dense", [9, 33, 0, 64, 65, 1, 31, 32] * 25, 384, 768, 200, True),
    ("two_per_cu_long_k", [63, 64, 49, 53, 64, 50, 64, 57] * 12, 1024, 768, 0, True),
    # tiles of 256 x 256 rows (no residual, K a multiple of 256, 1024 or more): remainders of
    # one and two such tiles, half tiles, and counts far from the mean
    ("wide_full", [200, 190, 225, 180] * 4, 1024, 4096, 0, True),
    ("wide_halves", [128, 127, 97, 64, 65, 96] * 4, 1024, 1536, 0, False),
    ("wide_uneven", [600, 0, 130, 129, 1, 512, 257, 200] * 3, 1280, 1536, 0, True),
    ("wide_one_expert", [13 * 256], 1024, 4096, 0, False),
    # the panel kernel's heights on more than two rounds of the chip, which the
    # tile kernel leaves to it
    ("panel64_edges", [63, 64, 65, 49] * 30, 256, 1152, 24, True),
    ("panel128_edges", [127, 128, 129, 97] * 25, 384, 1408, 40, True),
    ("panel192_edges", [191, 192, 193, 129] * 24, 256, 1536, 8, True),
    ("panel320_edges", [319, 320, 321, 289] * 12, 256, 1920, 16, True),
    ("panel320_one_expert", [6001], 256, 6016, 48, False),
    ("panel128_largest_table", [90, 70] * 50, 256, 1408, 144, True),
    ("panel128_dense", [150, 60, 100] * 32, 256, 1536, 200, True),
    ("panel320_dense", [300, 321] * 24, 256, 1920, 200, False),
    ("panel192_plain", [130, 97, 190, 200] * 25, 384, 1408, 0, True),
    # the tile kernel's ring of four slots with the A-scale ring, two passes of it,
    # and a table at K of no whole 256
    ("tile_plain_k512", [128, 120, 257, 0, 60], 512, 256, 0, True),
    ("tile_dense_k512", [100, 129, 33], 512, 256, 200, True),
    ("tile_table_k640", [63, 97, 200], 640, 128, 100, False),
    ("two_per_cu_table", [63, 64, 49, 33, 64, 50, 64, 17] * 25, 256, 768, 24, True),
]


@pytest.mark.parametrize("epi", [Q.QD_EPI_NONE, Q.QD_EPI_SWIGLU], ids=["plain", "swiglu"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_panel_gemm(case, epi):
    name, counts, K, N, Ks, gather = case
    E, R = len(counts), sum(counts)
    T = (R + 1) // 2 if gather else R
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    g = torch.Generator().manual_seed(zlib.crc32(name.encode()))
    x = torch.randn((T, K), generator=g)
    x[:, ::29] *= 20.0
    x = x.to(torch.bfloat16)
    wb = (torch.randn((E, N, K), generator=g) * 0.02).to(torch.bfloat16)
    tok = rng.integers(0, T, R).astype(np.int32) if gather else np.arange(R, dtype=np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    w, W = ops.quantize_weight(wb.to(DEV)), oracle_bank(wb)
    kind = Q.lib().moe_w4a4_grouped_gemm_kernel(R, N, K, E, Ks, epi, 0,
                                                int(w.scales_frag is not None)).decode()
    for k in ("panel64", "panel128", "panel192", "panel320", "tile", "wide"):
        assert kind == k or not name.startswith(k)
    assert kind == "panel64" or not name.startswith("two_per_cu")
    xg = x.to(DEV)
    xq, scores, ramax = ops.quantize_act(xg, rac=True)
    act = OR.rac_activation(np_bf16(x), Ks)
    assert_nvfp4_equal(xq, act["xq"], "xq")
    sel = rq = None
    if Ks:
        sel, rq, _, _ = ops.select_channels(xg, xq, Ks, scores, ramax)
        assert np.array_equal(sel.cpu().numpy(), act["sel"])
    out, amax = ops.grouped_gemm(xq, w, R, torch.from_numpy(tok).to(DEV) if gather else None,
                                 torch.from_numpy(offsets).to(DEV) if E > 1 else None, rq, sel,
                                 epi, want_amax=True)
    gu, mag = OL.w13_stage(act["xq"], act["rq"] if Ks else None, tok, offsets, W)
    if epi == Q.QD_EPI_SWIGLU:
        I = N // 2
        ref = OL.silu(gu[:, :I]) * gu[:, I:]
        mag = (np.abs(OL.silu(gu[:, :I])) * mag[:, I:] + 1.1 * np.abs(gu[:, I:]) * mag[:, :I])
    else:
        ref = gu
    check_close_bf16(np_bf16(out), ref, mag, name)
    assert amax.max().item() == np.max(np.abs(np_bf16(out)))


def test_panel_gemm_most_experts():
    """E = 1024, the last entry of the tile schedule: rows on the first, a
    middle and the last expert only."""
    E, K, N = 1024, 384, 128
    counts = np.zeros(E, np.int64)
    counts[[0, 517, 1023]] = (33, 70, 64)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offsets[-1])
    g = torch.Generator().manual_seed(7)
    x = torch.randn((R, K), generator=g).to(torch.bfloat16)
    wb = torch.zeros((E, N, K), dtype=torch.bfloat16)
    live = np.nonzero(counts)[0]
    for e in live:
        wb[e] = (torch.randn((N, K), generator=g) * 0.02).to(torch.bfloat16)
    w, W = ops.quantize_weight(wb.to(DEV)), oracle_bank(wb, live)
    xq, _, _ = ops.quantize_act(x.to(DEV))
    act = OR.rac_activation(np_bf16(x), 0)
    out, _ = ops.grouped_gemm(xq, w, R, None, torch.from_numpy(offsets).to(DEV))
    ref, mag = OL.w13_stage(act["xq"], None, np.arange(R), offsets, W)
    check_close_bf16(np_bf16(out), ref, mag, "E = 1024")


def test_wide_gemm_most_experts():
    """E = 1024 on the tiles of 256 x 256, about 200 rows each: the bits of the
    panel kernel, which weights without fragment-ordered scales take."""
    E, K, N = 1024, 1024, 256
    rng = np.random.default_rng(17)
    counts = rng.integers(190, 211, E)
    counts[:2] = (255, 0)
    counts[-1] = 256
    offsets = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).to(DEV)
    R = int(counts.sum())
    g = torch.Generator(device=DEV).manual_seed(17)
    x = torch.randn((R, K), generator=g, device=DEV).to(torch.bfloat16)
    wb = (torch.randn((E, N, K), generator=g, device=DEV) * 0.02).to(torch.bfloat16)
    xq, _, _ = ops.quantize_act(x)
    kernel = Q.lib().moe_w4a4_grouped_gemm_kernel
    assert [kernel(R, N, K, E, 0, 0, 0, f) for f in (1, 0)] == [b"wide", b"panel320"]
    out, amax = ops.grouped_gemm(xq, ops.quantize_weight(wb), R, None, offsets, want_amax=True)
    ref, _ = ops.grouped_gemm(xq, ops.quantize_weight(wb, frag_scales=False), R, None, offsets)
    assert torch.equal(out, ref)
    assert amax.max().item() == ref.float().abs().max().item()


@pytest.mark.parametrize("Ks", [0, 48, 200], ids=["plain", "compact", "dense"])
def test_panel_and_tile_kernels_agree(Ks):
    """The rows of a few experts in a small call (tile kernel) and among those of
    many (panel kernel): the same up to the order of the f32 sums, so within half a
    bf16 ulp of nearly the same value."""
    few, many, K, N = 4, 120, 512, 1536
    rng = np.random.default_rng(23)
    counts = rng.integers(100, 140, many)
    n = int(counts[:few].sum())
    offs = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).to(DEV)
    R = int(counts.sum())
    g = torch.Generator(device=DEV).manual_seed(23)
    x = torch.randn((R, K), generator=g, device=DEV)
    x[:, ::17] *= 20.0
    x = x.to(torch.bfloat16)
    w = ops.quantize_weight((torch.randn((many, N, K), generator=g, device=DEV) * 0.02)
                            .to(torch.bfloat16), frag_scales=False)
    v = ops.NVFP4Tensor(w.codes[:few], w.scales[:few], w.gscale[:few], few, N, K)
    kernel = Q.lib().moe_w4a4_grouped_gemm_kernel
    assert kernel(n, N, K, few, Ks, 0, 0, 0) == b"tile"
    assert kernel(R, N, K, many, Ks, 0, 0, 0).startswith(b"panel")
    xq, scores, ramax = ops.quantize_act(x, rac=True)
    sel = rq = None
    if Ks:
        sel, rq, _, _ = ops.select_channels(x, xq, Ks, scores, ramax)
    a, _ = ops.grouped_gemm(xq, v, n, None, offs[:few + 1].contiguous(), rq, sel)
    b, _ = ops.grouped_gemm(xq, w, R, None, offs, rq, sel)
    a, b = a.double(), b[:n].double()
    assert (a - b).norm() / b.norm() <= 2.0 ** -8


@pytest.mark.parametrize("Ks,n", [(24, 1), (250, 1), (24, 40)], ids=["tile", "tile_250", "panel"])
def test_panel_gemm_per_expert_sets(Ks, n):
    """One channel set per expert: the tile kernel, also above the panel kernel's
    largest table, and the panel kernel."""
    counts, K, N = [130, 0, 65, 33] * n, 512, 256 if n == 1 else 1152
    kind = Q.lib().moe_w4a4_grouped_gemm_kernel(sum(counts), N, K, len(counts), Ks, 0, 1, 1)
    assert kind.startswith(b"tile" if n == 1 else b"panel")
    E, R = len(counts), sum(counts)
    T = R // 2
    rng = np.random.default_rng(5)
    g = torch.Generator().manual_seed(5)
    x = torch.randn((T, K), generator=g)
    x[:, ::17] *= 20.0
    x = x.to(torch.bfloat16)
    wb = (torch.randn((E, N, K), generator=g) * 0.02).to(torch.bfloat16)
    tok = np.concatenate([np.sort(rng.integers(0, T, c)) for c in counts]).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    w, W = ops.quantize_weight(wb.to(DEV)), oracle_bank(wb)
    xg, tg, og = x.to(DEV), torch.from_numpy(tok).to(DEV), torch.from_numpy(offsets).to(DEV)
    xq, _, _ = ops.quantize_act(xg)
    sel, rq, rows, _, _ = ops.select_channels_per_expert(xg, xq, Ks, tg, og)
    act = OR.rac_activation_per_expert(np_bf16(x), Ks, tok, offsets)
    assert np.array_equal(sel.cpu().numpy(), act["sel_pe"])
    out, _ = ops.grouped_gemm_per_expert(xq, w, R, tg, og, rq, sel, rows)
    ref, mag = OL.w13_stage_per_expert(act["xq"], act["rq"], act["sel_pe"], tok, offsets, W)
    check_close_bf16(np_bf16(out), ref, mag, f"per-expert sets, K_s = {Ks}")


def test_panel_gemm_many_rows_of_one_expert():
    """Eight million rows on one expert (26,215 tiles): row i of the result is
    that of its token, on the W4A4, W4A16 and FP8 kernels alike."""
    R, T, K, N = 1 << 23, 997, 256, 128
    g = torch.Generator().manual_seed(11)
    x = torch.randn((T, K), generator=g).to(torch.bfloat16).to(DEV)
    wb = (torch.randn((1, N, K), generator=g) * 0.02).to(torch.bfloat16).to(DEV)
    tok = (torch.arange(R, device=DEV, dtype=torch.int64) % T).to(torch.int32)
    w = ops.quantize_weight(wb)
    xq, _, _ = ops.quantize_act(x)
    xc, xd = ops.fp8_quantize_rows(x)
    wc, wd = ops.fp8_quantize_rows(wb)
    w32 = ops.quantize_weight(wb[:, :32, :128].contiguous())
    x128 = x[:, :128].contiguous()
    for name, call in (("W4A4", lambda n, t: ops.grouped_gemm(xq, w, n, t)[0]),
                       ("W4A16", lambda n, t: ops.w4a16_grouped_gemm(x128, w32, n, t)),
                       ("FP8", lambda n, t: ops.fp8_grouped_gemm(xc, xd, wc, wd, n, t))):
        few = call(T, torch.arange(T, dtype=torch.int32, device=DEV))
        out = call(R, tok)
        for r0 in range(0, R, 1 << 20):
            t = tok[r0:r0 + (1 << 20)].long()
            assert torch.equal(out[r0:r0 + (1 << 20)], few[t]), f"{name}: rows {r0} on"


@pytest.mark.parametrize("Ks", [0, 16, 200], ids=["plain", "compact", "dense"])
def test_rows_past_4_gib_of_activations(Ks):
    """row_token names rows whose codes lie past 4 GiB of a larger matrix: what
    the same rows give on their own.  Two kernels, so two roundings of sums in
    another order: each within half a bf16 ulp of nearly the same value."""
    K, N, n, E = 256, 256, 300, 2
    A = 2 * 2 ** 32 // K + n
    g = torch.Generator().manual_seed(13)
    x = torch.randn((n, K), generator=g)
    x[:, ::17] *= 20.0
    xg = x.to(torch.bfloat16).to(DEV)
    w = ops.quantize_weight((torch.randn((E, N, K), generator=g) * 0.02).to(torch.bfloat16).to(DEV))
    xq, scores, ramax = ops.quantize_act(xg, rac=True)
    sel = rq = None
    if Ks:
        sel, rq, _, _ = ops.select_channels(xg, xq, Ks, scores, ramax)

    def far(t):
        big = ops.NVFP4Tensor.empty(1, A, K, DEV)
        big.codes.zero_()
        big.scales.zero_()
        big.codes[0, -n:] = t.codes[0]
        big.scales[0, -n:] = t.scales[0]
        big.gscale.copy_(t.gscale)
        return big

    tok = torch.arange(n, dtype=torch.int32, device=DEV)
    offs = torch.tensor([0, n // 2, n], dtype=torch.int32, device=DEV)
    near, _ = ops.grouped_gemm(xq, w, n, tok, offs, rq, sel)
    out, _ = ops.grouped_gemm(far(xq), w, n, tok + (A - n), offs, far(rq) if Ks else None, sel,
                              rq_sel=ops.gather_selected(rq, sel) if Ks else None)
    d = (out.double() - near.double()).norm() / near.double().norm()
    assert d <= 2.0 ** -8, float(d)
