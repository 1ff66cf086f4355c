"""Performance cases: the calls a user of this package makes, over the sizes they meet.

The NVFP4 W4A4 MoE layer with residual compensation is the product, so most
cases are one layer step at a batch size of serving (one token, decode batches,
a chunk between decode and prefill, prefill) and at the widths of this
repository's workloads; the others are the block entry point (norm and router
folded in), the trainer-side forward on the same weights, the FP8 layer and
the weight sync (quantising a bank after a training step).

`exact` restates each call in plain torch: the quantisers' decisions in the
float32 sequence that defines the formats, every contraction in float64.
"""

import math

import torch

from paper_2607_15810_amd import ops

DEV = "cuda"


def _layer(name, T, H, I, Ks, E=128, k=8, routing="normal", acts="normal"):
    return dict(name=name, kind="layer", T=T, H=H, E=E, k=k, I=I, Ks=Ks, routing=routing,
                acts=acts)


def listed():
    return [
        # one request decoding alone: launches and latency
        _layer("layer_t1_h2048", 1, 2048, 768, 64),
        # a decode batch, every expert touched
        _layer("layer_t256_h2048", 256, 2048, 768, 64),
        # a decode batch on one rank of a two-way tensor-parallel rollout:
        # half the expert width, which is no multiple of 256
        _layer("layer_t96_i384", 96, 2048, 384, 64),
        # decode with skewed expert popularity and heavy-tailed activations
        _layer("layer_zipf_t64_h4096", 64, 4096, 1536, 128, routing="zipf", acts="student_t3"),
        # a chunk of prompt tokens mixed with decode: more rows per expert than
        # a decode batch, far fewer than a prefill
        _layer("layer_t1000_h2048", 1000, 2048, 768, 64),
        # prefill, narrow and wide model
        _layer("layer_t8192_h2048", 8192, 2048, 768, 64),
        _layer("layer_t4096_h4096", 4096, 4096, 1536, 128),
        # prefill with half of the channels compensated
        _layer("layer_half_t2048_h2048", 2048, 2048, 768, 1024),
        # the layer fed from the hidden state (norm and router folded in), a
        # ragged prefill
        dict(name="block_t2000_h2048", kind="block", T=2000, H=2048, E=128, k=8, I=768, Ks=64),
        # the trainer's forward on the rollout's weights
        dict(name="w4a16_t4096_h2048", kind="w4a16", T=4096, H=2048, E=128, k=8, I=768),
        # the FP8 rollout's layer, prefill
        dict(name="fp8_t4096_h2048", kind="fp8", T=4096, H=2048, E=128, k=8, I=768),
        # weight sync: one layer's gate/up bank quantised after a training step
        dict(name="weights_e128_h2048", kind="weights", E=128, N=1536, K=2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer"] * 8 + ["block"] * 2 + ["w4a16", "fp8", "weights"])
    if kind == "weights":
        return dict(kind="weights", E=rng.choice([32, 48, 64, 96, 128]),
                    N=256 * rng.randint(3, 8), K=256 * rng.randint(4, 12))
    H = rng.choice([2048, 2048, 3072, 4096])
    I = rng.choice([384, 768, 1024, 1536])
    E = rng.choice([64, 128, 128])
    k = rng.choice([4, 8, 8])
    Ks = rng.choice([0, H // 32, H // 32, H // 32, H // 2])
    most = 4096 * 4096 * 1536 if kind in ("layer", "block") and Ks < H // 2 else 2048 * 4096 * 1536
    top = min(8192, most // (H * I))
    T = _log_int(rng, 1 if kind in ("layer", "block") else 16, top)
    T += T % 2 == 0 and rng.random() < 0.5       # half of the even draws made odd
    c = dict(kind=kind, T=min(T, top), H=H, E=E, k=k, I=I)
    if kind in ("layer", "block"):
        c["Ks"] = Ks
    if kind == "layer":
        c["routing"] = rng.choice(["normal", "normal", "zipf"])
        c["acts"] = rng.choice(["normal", "normal", "student_t3"])
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed, device=DEV):
    g = torch.Generator(device=device)
    g.manual_seed(1000003 * (int(seed) + 1))
    return g


def _acts(c, g):
    """Activations with a few outlier channels, or heavy-tailed ones."""
    T, H = c["T"], c["H"]
    x = torch.randn((T, H), generator=g, device=DEV)
    if c.get("acts", "normal") == "student_t3":
        d = torch.zeros((T, H), device=DEV)
        for _ in range(3):
            d += torch.randn((T, H), generator=g, device=DEV).square()
        x /= torch.sqrt(d / 3.0).clamp_min(1e-3)
    else:
        n = max(1, round(0.01 * H))
        ch = torch.randperm(H, generator=g, device=DEV)[:n]
        x[:, ch] *= 50.0 if H >= 4096 else 20.0
    return x.to(torch.bfloat16)


def _logits(c, g, device=DEV):
    T, E = c["T"], c["E"]
    if c.get("routing", "normal") != "zipf":
        return torch.randn((T, E), generator=g, device=device)
    p = torch.arange(1, E + 1, device=device, dtype=torch.float32).pow(-1.2)
    base = torch.log(p / p.sum())[torch.randperm(E, generator=g, device=device)]
    u = torch.rand((T, E), generator=g, device=device).clamp(1e-7, 1 - 1e-7)
    return base - torch.log(-torch.log(u))


def _bank(E, N, K, g):
    w = torch.empty((E, N, K), dtype=torch.bfloat16, device=DEV)
    for e in range(0, E, 16):
        n = min(16, E - e)
        w[e:e + n] = torch.randn((n, N, K), generator=g, device=DEV) * 0.02
    return w


def _inputs(c, seed):
    """The seeded inputs of a case, as bf16 / f32 tensors on the GPU."""
    g = _gen(seed)
    if c["kind"] == "weights":
        return dict(w=_bank(c["E"], c["N"], c["K"], g))
    d = dict(x=_acts(c, g))
    if c["kind"] == "block":
        d["gamma"] = (1.0 + 0.1 * torch.randn(c["H"], generator=g, device=DEV)).to(torch.bfloat16)
        d["router"] = (0.02 * torch.randn((c["E"], c["H"]), generator=g, device=DEV)).to(
            torch.bfloat16)
    else:
        d["logits"] = _logits(c, g)
    d["w13"] = _bank(c["E"], 2 * c["I"], c["H"], g)
    d["w2"] = _bank(c["E"], c["H"], c["I"], g)
    return d


def prepare(case, seed):
    c, d = case, _inputs(case, seed)
    kind = c["kind"]
    if kind == "weights":
        return dict(kind=kind, w=d["w"])
    if kind == "fp8":
        w13, s13 = ops.fp8_quantize_rows(d["w13"])
        w2, s2 = ops.fp8_quantize_rows(d["w2"])
        lay = ops.FP8MoELayer(w13, s13, w2, s2, c["T"], c["k"])
        return dict(kind=kind, layer=lay, args=(d["x"], d["logits"]))
    w13, w2 = ops.quantize_weight(d["w13"]), ops.quantize_weight(d["w2"])
    if kind == "w4a16":
        lay = ops.W4A16MoELayer(w13, w2, c["k"])
        return dict(kind=kind, layer=lay, args=(d["x"], d["logits"]))
    if kind == "block":
        lay = ops.MoEBlock(w13, w2, c["T"], c["k"], c["Ks"], d["gamma"], d["router"])
        return dict(kind=kind, layer=lay, args=(d["x"],))
    lay = ops.MoELayer(w13, w2, c["T"], c["k"], c["Ks"])
    return dict(kind=kind, layer=lay, args=(d["x"], d["logits"]))


def run(state):
    if state["kind"] == "weights":
        q = ops.quantize_weight(state["w"])
        return dict(codes=q.codes, scales=q.scales, gscale=q.gscale, scales_frag=q.scales_frag)
    return state["layer"](*state["args"])


# ------------------------------------------------------------------ work

def _touched(c):
    """Experts with at least one row, for one draw of the routing."""
    lg = _logits(dict(c, T=min(c["T"], 2048)), _gen(0, "cpu"), "cpu")
    return int(torch.unique(torch.topk(lg, c["k"], dim=1).indices).numel())


def work(case):
    c = case
    if c["kind"] == "weights":
        n = c["E"] * c["N"] * c["K"]
        return dict(bytes=n * (2 + 0.5625 + 0.0625), flops=0)
    T, H, I, E, k = c["T"], c["H"], c["I"], c["E"], c["k"]
    R, Ks = T * k, c.get("Ks", 0)
    per = 1.0 if c["kind"] == "fp8" else 0.5625
    nbytes = _touched(c) * 3 * I * H * per + 2 * T * H * 2
    flops = 2 * R * 3 * I * H + 2 * R * 2 * I * Ks
    if c["kind"] == "block":
        nbytes += 2 * E * H
        flops += 2 * T * H * E
    else:
        nbytes += 4 * T * E
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    if case["kind"] == "weights":
        return "exact"
    # about four times what the calls differ from `exact` by: the rounding of
    # bf16 results, and where a sum in another order turns a rounding of h or
    # x, the quantised value after it
    return {"block": dict(rel=1e-2, max=0.8), "fp8": dict(rel=1.2e-2, max=0.5)}.get(
        case["kind"], dict(rel=7e-3, max=0.32))


# ------------------------------------------------------------------ the same in 64 bits

_E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _e2m1_index(a):
    """Nearest E2M1 magnitude, ties to the even code, saturating at 6."""
    i = (a > 0.25).to(torch.uint8)
    for edge, closed in ((0.75, True), (1.25, False), (1.75, True), (2.5, False), (3.5, True),
                         (5.0, False)):
        i += (a >= edge) if closed else (a > edge)
    return i


def _quant(x):
    """NVFP4 quantisation of a float32 matrix with one tensor scale: (code
    index, sign, block scale byte, block scale value, s_enc, s_dec)."""
    rows, cols = x.shape
    one = torch.ones((), device=DEV)
    amax = x.abs().max()
    s_enc = (2688.0 * one) / amax
    s_dec = one / s_enc
    if not amax >= 2.0 ** -100:
        s_enc, s_dec = one, one
    b = x.view(rows, cols // 16, 16)
    t = (b.abs().amax(-1) / (6.0 * one)) * s_enc
    f8 = torch.clamp(t, max=448.0).to(torch.float8_e4m3fn)
    sv = f8.float()
    if not amax >= 2.0 ** -100:
        sv = torch.zeros_like(sv)
    enc = torch.where(sv > 0, s_enc / torch.where(sv > 0, sv, one), torch.zeros_like(sv))
    idx = _e2m1_index((b * enc.unsqueeze(-1)).abs())
    return idx, torch.signbit(b), f8.view(torch.uint8), sv, s_enc, s_dec


def _values(q, shape):
    """Unscaled values e2m1 * e4m3 (exact in float32)."""
    lut = torch.tensor(_E2M1, device=DEV)
    v = lut[q[0].long()] * q[3].unsqueeze(-1)
    return torch.where(q[1], -v, v).view(shape)


def _bf16(v):
    """Round float64 to bf16 (the format the layer keeps h and z in)."""
    return v.float().to(torch.bfloat16).double()


def _act_operand(x, Ks):
    """The compensated activation x_hat - M_S Q_A(x_hat - x) in float64."""
    q = _quant(x)
    v = _values(q, x.shape)
    xt = v.double() * q[5].double()
    if Ks == 0:
        return xt
    r = v * q[5] - x
    e = math.frexp(float(x.abs().max()))[1]
    score = torch.trunc((r * r).double() * 2.0 ** (36 - 2 * e)).to(torch.int64).sum(0)
    sel = torch.sort(score, descending=True, stable=True).indices[:Ks]
    rq = _quant(r)
    rv = _values(rq, r.shape).double() * rq[5].double()
    xt[:, sel] -= rv[:, sel]
    return xt


def _fp8_rows(x):
    m = x.abs().amax(-1, keepdim=True)
    one = torch.ones((), device=DEV)
    enc = torch.where(m > 0, (448.0 * one) / torch.where(m > 0, m, one), one)
    v = torch.clamp((x * enc).abs(), max=448.0).to(torch.float8_e4m3fn).double()
    return torch.where(torch.signbit(x), -v, v) * (one / enc).double()


def _weight(kind, w):
    """One expert's dequantised weights in float64."""
    if kind == "fp8":
        return _fp8_rows(w.float())
    q = _quant(w.float())
    return _values(q, w.shape).double() * q[5].double()


def exact(case, seed):
    c, d = case, _inputs(case, seed)
    kind = c["kind"]
    if kind == "weights":
        E, N, K = c["E"], c["N"], c["K"]
        gs = torch.empty((E, 2), dtype=torch.float64, device=DEV)
        for e in range(E):
            amax = d["w"][e].abs().max().double()
            gs[e, 0] = 2688.0 / amax
            gs[e, 1] = amax / 2688.0
        return dict(codes=None, scales=None, gscale=gs, scales_frag=None)
    T, H, E, k, I = c["T"], c["H"], c["E"], c["k"], c["I"]
    x = d["x"].double()
    if kind == "block":
        x = _bf16(x / torch.sqrt(x.square().mean(-1, keepdim=True) + 1e-6) * d["gamma"].double())
        logits = (x @ d["router"].double().t()).float()
    else:
        logits = d["logits"]
    top, ids = torch.sort(logits, dim=1, descending=True, stable=True)
    ids = ids[:, :k]
    wts = torch.softmax(top[:, :k].double(), dim=1)
    if kind == "w4a16":
        a = x
    elif kind == "fp8":
        a = _fp8_rows(x.float())
    else:
        a = _act_operand(x.float(), c["Ks"])
    rows = [torch.nonzero(ids == e) for e in range(E)]
    h = torch.zeros((T * k, I), dtype=torch.float64, device=DEV)
    for e in range(E):
        t, s = rows[e][:, 0], rows[e][:, 1]
        if t.numel() == 0:
            continue
        gu = a[t] @ _weight(kind, d["w13"][e]).t()
        g, u = gu[:, :I], gu[:, I:]
        h[t * k + s] = _bf16(g / (1.0 + torch.exp(-g)) * u)
    if kind == "fp8":
        h = _fp8_rows(h.float())
    elif kind != "w4a16":
        h = _act_operand(h.float(), 0)
    z = torch.zeros((T * k, H), dtype=torch.float64, device=DEV)
    for e in range(E):
        r = rows[e][:, 0] * k + rows[e][:, 1]
        if r.numel():
            z[r] = _bf16(h[r] @ _weight(kind, d["w2"][e]).t())
    return (z.view(T, k, H) * wts.unsqueeze(-1)).sum(1)
