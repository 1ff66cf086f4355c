"""GPU parity of the grouped prefill GEMM over unpacked activations (W4A16 and
FP8) at the edges of its tiles: row counts around its 32-row fragments and
around each tile height (64, 128, 192, 320 rows), widths that are no multiple
of its 256 weight rows (a last 32-row fragment, a half SwiGLU fragment), the
smallest K, and the largest expert count of its schedule.

Against the oracle's float64 contraction of the same operands, with the
tolerance every stage of either layer has."""

import zlib

import numpy as np
import pytest
import torch

from oracle import fp8 as OF, layer as OL, w4a16 as OW
from paper_2607_15810_amd import ops
from paper_2607_15810_amd import quads as Q

from helpers import check_close_bf16, np_bf16, oracle_bank

pytestmark = pytest.mark.gpu

DEV = "cuda"
EPIS = [Q.QD_EPI_NONE, Q.QD_EPI_SWIGLU]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q.lib()
    yield


def _inputs(name, counts, K, N, gather):
    E, R = len(counts), sum(counts)
    T = (R + 1) // 2 if gather else R
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    g = torch.Generator().manual_seed(zlib.crc32(name.encode()))
    x = torch.randn((T, K), generator=g)
    x[:, ::29] *= 20.0
    w = (torch.randn((E, N, K), generator=g) * 0.02).to(torch.bfloat16)
    tok = rng.integers(0, T, R).astype(np.int32) if gather else None
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    tg = torch.from_numpy(tok).to(DEV) if gather else None
    return x.to(torch.bfloat16), w, tok, offsets, tg, torch.from_numpy(offsets).to(DEV)


def _reference(gu, mag, epi):
    if epi == Q.QD_EPI_NONE:
        return gu, mag
    I = gu.shape[1] // 2
    s = OL.silu(gu[:, :I])
    return s * gu[:, I:], np.abs(s) * mag[:, I:] + 1.1 * np.abs(gu[:, I:]) * mag[:, :I]


W4A16 = [
    # name, rows per expert, K, N, gathered rows
    ("two_stages", [1, 31, 32, 33, 0, 5], 128, 256, True),
    ("odd_stages", [63, 64, 65, 0], 320, 32, False),
    ("half_fragment", [70, 64, 65, 96], 192, 96, True),
    ("around_128", [127, 128, 129, 97], 512, 288, True),
    ("around_192", [191, 192, 193, 129], 256, 384, True),
    ("around_320", [319, 320, 321, 289], 512, 256, False),
    ("two_tiles", [640, 641, 1, 330], 256, 544, True),
    ("one_expert", [333], 384, 256, False),
    ("one_row", [1], 768, 256, False),
    ("one_stage", [40, 90], 64, 256, True),             # K of one stage: the other kernel
    ("full_tiles", [100, 128, 64, 1], 2048, 256, True), # full tiles in one round: the other one
]


@pytest.mark.parametrize("epi", EPIS, ids=["plain", "swiglu"])
@pytest.mark.parametrize("case", W4A16, ids=[c[0] for c in W4A16])
def test_w4a16_gemm(case, epi):
    name, counts, K, N, gather = case
    x, wb, tok, offsets, tg, og = _inputs(name, counts, K, N, gather)
    w, W = ops.quantize_weight(wb.to(DEV)), oracle_bank(wb)
    R = sum(counts)
    out = ops.w4a16_grouped_gemm(x.to(DEV), w, R, tg, og if len(counts) > 1 else None, epi)
    ref, mag = _reference(*OW.grouped_gemm(np_bf16(x), tok, offsets, W), epi)
    check_close_bf16(np_bf16(out), ref, mag, name)


@pytest.mark.parametrize("epi", EPIS, ids=["plain", "swiglu"])
@pytest.mark.parametrize("case", [c for c in W4A16 if c[0] != "one_stage"] +
                         [("long_k", [3, 40, 0, 97], 2112, 96, True)],
                         ids=lambda c: c[0])
def test_w4a16_order_of_sums(case, epi):
    """The bits of a result do not depend on which of the two kernels ran: the
    general one takes over where the activations pass 4 GiB, declared here for
    a matrix whose later rows no token names."""
    name, counts, K, N, _ = case
    x, wb, tok, offsets, tg, og = _inputs(name, counts, K, N, True)
    w, R, E = ops.quantize_weight(wb.to(DEV)), sum(counts), len(counts)
    xg = x.to(DEV)
    outs = []
    for a_rows in (len(x), 2 ** 32 // (2 * K) + 1):
        out = torch.empty((R, N // 2 if epi else N), dtype=torch.bfloat16, device=DEV)
        Q.call("moe_w4a16_grouped_gemm", xg.data_ptr(), a_rows, tg.data_ptr(), og.data_ptr(), E, R,
               ops._nv(w), epi, out.data_ptr(), ops._stream())
        outs.append(out)
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


def _height_case(mean):
    """128 experts of about `mean` rows each, N = 1536, K = 256: the tile height
    follows the mean (test_panel_schedule.py); counts around it, among them none, one
    row and a tile of every other height."""
    E, K, N = 128, 256, 1536
    rng = np.random.default_rng(mean)
    counts = rng.integers(mean - 6, mean + 7, E)
    counts[[3, 40, 90, 127]] = (0, 1, 2 * mean, mean + mean - 1)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offsets[-1])
    T = R // 4
    tok = rng.integers(0, T, R).astype(np.int32)
    g = torch.Generator().manual_seed(mean)
    x = torch.randn((T, K), generator=g)
    x[:, ::29] *= 20.0
    wb = (torch.randn((E, N, K), generator=g) * 0.02).to(torch.bfloat16)
    return E, K, N, R, counts, offsets, tok, x.to(torch.bfloat16), wb


@pytest.mark.parametrize("epi", EPIS, ids=["plain", "swiglu"])
@pytest.mark.parametrize("mean", [30, 88, 145, 250])
def test_w4a16_heights(mean, epi):
    """Every tile height on several rounds of the chip: the general kernel's bits."""
    E, K, N, R, _, offsets, tok, x, wb = _height_case(mean)
    w, xg = ops.quantize_weight(wb.to(DEV)), x.to(DEV)
    tg, og = torch.from_numpy(tok).to(DEV), torch.from_numpy(offsets).to(DEV)
    outs = []
    for a_rows in (len(x), 2 ** 32 // (2 * K) + 1):
        out = torch.empty((R, N // 2 if epi else N), dtype=torch.bfloat16, device=DEV)
        Q.call("moe_w4a16_grouped_gemm", xg.data_ptr(), a_rows, tg.data_ptr(), og.data_ptr(), E, R,
               ops._nv(w), epi, out.data_ptr(), ops._stream())
        outs.append(out)
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


@pytest.mark.parametrize("epi", EPIS, ids=["plain", "swiglu"])
@pytest.mark.parametrize("mean", [30, 88, 145, 250])
def test_fp8_heights(mean, epi):
    """The same for FP8, against the oracle on six of the experts."""
    E, K, N, R, counts, offsets, tok, x, wb = _height_case(mean)
    ac, ad = ops.fp8_quantize_rows(x.to(DEV))
    wc, wd = ops.fp8_quantize_rows(wb.to(DEV))
    out = np_bf16(ops.fp8_grouped_gemm(ac, ad, wc, wd, R, torch.from_numpy(tok).to(DEV),
                                       torch.from_numpy(offsets).to(DEV), epi))
    pick = [0, 40, 64, 90, 101, 127]
    rows = np.concatenate([np.arange(offsets[e], offsets[e + 1]) for e in pick])
    offs = np.concatenate([[0], np.cumsum(counts[pick])]).astype(np.int32)
    bank = OF.quantize_bank(wb[pick].float().numpy())
    gu, mag = OF.grouped_gemm(*OF.quantize_rows(np_bf16(x)), tok[rows], offs, bank)
    ref, mag = _reference(gu, mag, epi)
    check_close_bf16(out[rows], ref, mag, f"{mean} rows per expert", floor=2.0 ** -13)


def test_w4a16_swiglu_range():
    """The SwiGLU epilogue over gates from deep underflow to overflow, zero and
    the non-finite ones (its first 32 rows hold moderate gates only): one weight of 6
    in every row, so that g = u = 6 x exactly."""
    K, N = 128, 64
    v = torch.cat([torch.linspace(-13.0, 13.0, 32), torch.tensor([0.0, -0.0, 1e-3, -1e-3, 0.7, -0.7, 5.0, -5.0, 20.0, -20.0, 79.0, -79.0, 81.0,
                      -81.0, 88.0, -88.0, 89.0, -89.0, 200.0, -200.0, 1e4, -1e4, 1e18, -1e18,
                      float("inf"), float("nan")])])
    x = torch.zeros((len(v), K))
    x[:, 0] = v
    x = x.to(torch.bfloat16)
    w = torch.zeros((1, N, K))
    w[:, :, 0] = 6.0                        # quantises exactly
    q = ops.quantize_weight(w.to(torch.bfloat16).to(DEV))
    out = ops.w4a16_grouped_gemm(x.to(DEV), q, len(v), None, None, Q.QD_EPI_SWIGLU)
    z = x[:-2, 0].double().numpy() * 6.0
    with np.errstate(over="ignore"):
        ref = z / (1.0 + np.exp(-z)) * z
    assert np.abs(z[:32]).max() < 80.0
    got = np_bf16(out)[:, 0].astype(np.float64)
    assert np.isnan(got[-1])
    bf = torch.from_numpy(ref.astype(np.float32)).to(torch.bfloat16).double().numpy()
    # below 2^-126 f32 may flush: 1e-37 covers it
    assert np.all(np.abs(got[:-2] - bf) <= 2.0 ** -8 * np.abs(bf) + 1e-37), (got[:-2], bf)


FP8 = [
    # name, rows per expert, K, N, gathered rows (above 48 rows per expert on average, but
    # for the last)
    ("two_stages", [1, 131, 32, 133, 0, 95], 256, 256, True),
    ("odd_stages", [63, 64, 65, 0, 90], 384, 256, False),
    ("around_128", [127, 128, 129, 97], 512, 768, True),
    ("around_192", [191, 192, 193, 129], 256, 384, True),
    ("around_320", [319, 320, 321, 289], 512, 256, False),
    ("two_tiles", [640, 641, 1, 330], 256, 512, True),
    ("one_expert", [333], 384, 256, False),
    ("half_stage", [100, 90], 320, 256, True),          # K of whole and a half: the other kernel
    # the other kernel's passes of 32 rows: K of whole and a half stages, a short K and
    # few tiles, and a long K
    ("passes_half_stage", [1, 31, 32, 33, 0, 48], 320, 256, True),
    ("passes_short_k", [1, 16, 0, 33, 5], 384, 512, False),
    ("passes_few_tiles", [31, 0, 1, 9], 1024, 768, True),
    ("passes_long_k", [1, 16, 31, 0, 9], 4096, 256, True),
]


@pytest.mark.parametrize("epi", EPIS, ids=["plain", "swiglu"])
@pytest.mark.parametrize("case", FP8, ids=[c[0] for c in FP8])
def test_fp8_gemm(case, epi):
    name, counts, K, N, gather = case
    x, wb, tok, offsets, tg, og = _inputs(name, counts, K, N, gather)
    ac, ad = ops.fp8_quantize_rows(x.to(DEV))
    wc, wd = ops.fp8_quantize_rows(wb.to(DEV))
    R = sum(counts)
    out = ops.fp8_grouped_gemm(ac, ad, wc, wd, R, tg, og if len(counts) > 1 else None, epi)
    bank = OF.quantize_bank(wb.float().numpy())
    gu, mag = OF.grouped_gemm(*OF.quantize_rows(np_bf16(x)), tok, offsets, bank)
    ref, mag = _reference(gu, mag, epi)
    check_close_bf16(np_bf16(out), ref, mag, name, floor=2.0 ** -13)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("K", [8, 504, 512, 520, 4096, 4104, 13, 1001])
def test_fp8_rows_exact(K, dtype):
    """Row codes bit for bit at the edges of the 8-element groups, 512-element
    passes and the 4096 elements kept in registers (13 and 1001: the general
    kernel), with non-finite elements."""
    g = torch.Generator().manual_seed(K)
    x = torch.randn((7, K), generator=g) * torch.exp(3.0 * torch.randn((7, K), generator=g))
    x[1] = 0.0
    x[2] *= -1e-30
    x[3, K // 2] = float("inf")
    x[4, K - 1] = float("nan")
    x = x.to(dtype)
    codes, dec = ops.fp8_quantize_rows(x.to(DEV))
    fin = [0, 1, 2, 5, 6]
    rc, rd = OF.quantize_rows(x.float().numpy()[fin])
    assert np.array_equal(codes.cpu().numpy()[fin], rc)
    assert np.array_equal(dec.cpu().numpy()[fin].view(np.uint32), rd.view(np.uint32))
    c = codes.cpu().numpy()
    # an infinite amax: scale 0, the element itself saturates, the rest is +-0
    assert c[3, K // 2] & 0x7F == 0x7E and not np.any(np.delete(c[3], K // 2) & 0x7F)
    # NaN is left out of the amax and saturates
    assert c[4, K - 1] & 0x7F == 0x7E


def test_fp8_rows_thresholds():
    """Every value of E4M3, every midpoint between two and its f32 neighbours."""
    grid = np.concatenate([np.arange(0, 9) * 2.0 ** -9,
                           [(8 + m) * 2.0 ** (e - 3) for e in range(-6, 9) for m in range(8)]])
    grid = np.unique(grid[grid <= 448.0]).astype(np.float32)
    mid = ((grid[1:] + grid[:-1]) / 2).astype(np.float32)
    v = np.concatenate([grid, mid, np.nextafter(mid, np.float32(0)),
                        np.nextafter(mid, np.float32(1e9)), [448.0] * 8]).astype(np.float32)
    v = np.concatenate([v, -v])
    v = v[:len(v) // 8 * 8]
    v[0] = 448.0                                   # amax 448: the row's scale is 1
    codes, _ = ops.fp8_quantize_rows(torch.from_numpy(v[None]).to(DEV))
    assert np.array_equal(codes.cpu().numpy(), OF.quantize_rows(v[None])[0])


def test_most_experts():
    """E = 1024, the last entry of the tile schedule: rows on the first, a
    middle and the last expert only."""
    E, K, N = 1024, 128, 128
    counts = np.zeros(E, np.int64)
    counts[[0, 517, 1023]] = (33, 70, 64)
    x, wb, tok, offsets, tg, og = _inputs("most", counts.tolist(), K, N, True)
    w = ops.quantize_weight(wb.to(DEV))
    W = oracle_bank(wb)
    out = ops.w4a16_grouped_gemm(x.to(DEV), w, int(counts.sum()), tg, og)
    ref, mag = OW.grouped_gemm(np_bf16(x), tok, offsets, W)
    check_close_bf16(np_bf16(out), ref, mag, "most experts")
