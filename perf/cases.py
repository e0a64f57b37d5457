"""Timing cases of the integer hot path: what a program that serves or
calibrates a fully quantized vision transformer asks of this library, through
`paper_2111_13824_amd`.

Every case has a "kind":

  ln      one PTF LayerNorm of int8 activations [T, C];
  head    Log-Int-Softmax of int32 logits [G, Lq, Lk] and the BitShift product
          with V [G, Lk, d], fused;
  qk      attention from int8 Q [G, Lq, dk], K [G, Lk, dk] and V [G, Lk, d],
          and its int32 result requantized for the next layer;
  maps    the attention maps themselves (codes of 4 or 8 bits, stored), then
          their product with V: the 8/8/8 setting, or maps kept for inspection;
  calib   PTF calibration of a float tensor [T, C] and its quantization;
  block   the integer steps around one attention layer, in order: LayerNorm,
          attention from Q, K and V, requantization.

`prepared` cases hold validated calls (prepare=True), as a low-latency serving
loop does; the others call the functions directly and let them allocate.

The listed sizes are those of the models this repository is measured on: DeiT-T
(batch 1) and DeiT-S (batch 8), ViT-B/16 at 224 px (batch 64), ViT-L/16 at
384 px (batch 16) and Swin-S (batch 32), whose patch merging normalizes rows of
up to 1536 channels.  draw() spreads over other batches, widths, resolutions
and head sizes, ragged ones among them.

Values follow the statistics of those models: LayerNorm inputs with per-channel
spreads log-uniform on [0.05, 2.5] (some channels 40 times the median), logits
of a normal distribution with a deviation of 3 at the logit scale, Q and K
rounded normal, V uniform over int8.
"""
from __future__ import annotations

import math

import torch

import paper_2111_13824_amd as fq

DEV = "cuda"
S10 = 2.0 ** -10


def listed():
    return [
        # The smallest call: one image through a DeiT-T attention layer, three
        # short launches in a serving loop; latency is all that counts.
        dict(name="block_deit_tiny_b1", kind="block", T=197, C=192, G=3, L=197, d=64,
             prepared=True),
        # Small-batch serving of DeiT-S: 48 attention units on 256 CUs.
        dict(name="head_deit_small_b8", kind="head", G=48, Lq=197, Lk=197, d=64, bits=4, Hb=0,
             zp_v=0, s_logit=S10, prepared=True),
        # LayerNorm of ViT-B/16 at a throughput batch.
        dict(name="ln_vit_base_b64", kind="ln", T=12608, C=768, K=3, bits=8, prepared=False),
        # LayerNorm of Swin-S's first stage: many short rows.
        dict(name="ln_swin_small_b32", kind="ln", T=100352, C=96, K=3, bits=8, prepared=False),
        # The norm of Swin-S's last patch merging (4 x 384 channels): few wide rows.
        dict(name="ln_swin_merge_b32", kind="ln", T=1568, C=1536, K=3, bits=8, prepared=False),
        # Fused attention of ViT-B/16 at a throughput batch.
        dict(name="head_vit_base_b64", kind="head", G=768, Lq=197, Lk=197, d=64, bits=4, Hb=0,
             zp_v=0, s_logit=S10, prepared=False),
        # Long rows: ViT-L/16 at 384 px.
        dict(name="head_vit_large_b16", kind="head", G=256, Lq=577, Lk=577, d=64, bits=4, Hb=0,
             zp_v=0, s_logit=S10, prepared=False),
        # Window attention of Swin-S with its relative-position bias.
        dict(name="head_swin_small_b32", kind="head", G=6144, Lq=49, Lk=49, d=32, bits=4, Hb=3,
             zp_v=0, s_logit=S10, prepared=False),
        # Integer-only attention from Q and K, then the next layer's input.
        dict(name="qk_vit_base_b64", kind="qk", G=768, Lq=197, Lk=197, dk=64, d=64, bits=4, Hb=0,
             zp=0, s_logit=S10, prepared=False),
        dict(name="qk_vit_large_b16", kind="qk", G=256, Lq=577, Lk=577, dk=64, d=64, bits=4, Hb=0,
             zp=0, s_logit=S10, prepared=False),
        # 8/8/8: 8-bit attention maps, then their product in int64.
        dict(name="maps8_vit_base_b64", kind="maps", G=768, Lq=197, Lk=197, d=64, bits=8, zp_v=0,
             s_logit=S10, prepared=False),
        # Post-training calibration of one activation tensor and its quantization.
        dict(name="calib_vit_base_b64", kind="calib", T=12608, C=768, K=3, bits=8,
             prepared=False),
    ]


# ---------------------------------------------------------------------------
# Drawn cases
# ---------------------------------------------------------------------------

# Model and patch-merging widths; a drawn width is one of them or any number
# of channels in the same range (a pruned model).
WIDTHS = (96, 128, 192, 256, 320, 384, 448, 512, 576, 640, 768, 896, 1024, 1152, 1280, 1408, 1536)
# Tokens of square images with and without a class token, and Swin windows.
SEQS = (49, 50, 64, 65, 144, 145, 196, 197, 256, 257, 324, 325, 400, 401, 576, 577)


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng):
    return rng.choice(WIDTHS) if rng.random() < 0.7 else rng.randint(96, 1536)


def _seq(rng, hi=640):
    return rng.choice(SEQS) if rng.random() < 0.6 else _log(rng, 16, hi)


def draw(rng):
    kind = rng.choice(("ln", "ln", "head", "head", "qk", "maps", "calib", "block"))
    if kind == "ln":
        C = _width(rng)
        T = _log(rng, 64, min(100352, 9_600_000 // C))
        return dict(kind=kind, T=T, C=C, K=rng.choice((3, 3, 3, 2, 4)),
                    bits=rng.choice((8, 8, 8, 6, 4)), prepared=T * C < 1_000_000)
    if kind == "calib":
        C = _width(rng)
        T = _log(rng, 64, min(100352, 9_600_000 // C))
        return dict(kind=kind, T=T, C=C, K=rng.choice((3, 3, 3, 2, 4)),
                    bits=rng.choice((8, 8, 8, 6, 4)), prepared=T * C < 1_000_000)
    if kind == "block":
        L, H = _seq(rng), rng.choice((3, 6, 12))
        B = _log(rng, 1, max(1, 4_000_000 // (H * L * L)))
        return dict(kind=kind, T=B * L, C=64 * H, G=B * H, L=L, d=64, prepared=True)
    # scales of the float and (the finest) the integer path
    s_logit = rng.choice((S10, S10, S10, S10, 2.0 ** -8, 2.0 ** -12))
    if kind == "qk":
        L = _seq(rng)
        dk = rng.choice((32, 64))
        H = rng.choice((3, 6, 12, 16))
        most = 20_000_000 if s_logit > 5e-4 else 10_000_000
        G = H * _log(rng, 1, max(1, most // (H * L * L)))
        return dict(kind=kind, G=G, Lq=L, Lk=L, dk=dk, d=dk, bits=rng.choice((4, 4, 4, 3)),
                    Hb=H if rng.random() < 0.3 else 0, zp=rng.choice((0, rng.randint(-20, 20))),
                    s_logit=s_logit, prepared=G * L * L < 1_000_000)
    # a class-attention layer has fewer queries than keys; images of up to
    # 512 px have up to 1025 tokens
    Lk = _seq(rng, 1025)
    Lq = Lk if rng.random() < 0.8 else rng.randint(1, Lk)
    H = rng.choice((3, 6, 12, 16))
    most = 20_000_000 if s_logit > 5e-4 and Lk <= 640 else 8_000_000
    G = H * _log(rng, 1, max(1, most // (H * Lq * Lk)))
    d = rng.choice((32, 64, 64, 64, 48, 80))
    small = G * Lq * Lk < 1_000_000
    if kind == "head":
        return dict(kind=kind, G=G, Lq=Lq, Lk=Lk, d=d, bits=rng.choice((4, 4, 4, 3)),
                    Hb=H if rng.random() < 0.3 else 0, zp_v=rng.choice((0, rng.randint(-20, 20))),
                    s_logit=s_logit, prepared=small)
    return dict(kind=kind, G=G, Lq=Lq, Lk=Lk, d=min(d, 64), bits=rng.choice((4, 8, 8)),
                zp_v=rng.choice((0, rng.randint(-20, 20))), s_logit=s_logit, prepared=small)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _int8(g, lo, hi, *shape):
    return torch.randint(lo, hi + 1, shape, generator=g, device=DEV, dtype=torch.int8)


def _activations(g, T, C):
    """Float activations with strong inter-channel variation, [T, C]."""
    u = torch.rand(C, generator=g, device=DEV)
    spread = torch.exp(math.log(0.05) + u * math.log(2.5 / 0.05))
    spread[torch.randperm(C, generator=g, device=DEV)[:max(1, C // 96)]] = 40 * spread.median()
    return _normal(g, T, C) * spread


def _ln_inputs(g, T, C, K, bits):
    """A PTF-quantized tensor: the layer-wise grid over all of x, each channel
    on the smallest power-of-two factor that holds it."""
    x = _activations(g, T, C)
    levels = 2 ** bits - 1
    lo, hi = x.min(), x.max()
    unit = (hi - lo) / levels / 2 ** K
    zp = torch.round(-lo / (2 ** K * unit)).clamp(0, levels)
    cmin, cmax = x.amin(0), x.amax(0)
    alpha = torch.full((C,), K, device=DEV, dtype=torch.int64)
    for a in range(K, -1, -1):
        step = 2 ** a * unit
        fits = (torch.round(cmin / step) + zp >= 0) & (torch.round(cmax / step) + zp <= levels)
        alpha[fits] = a
    half = 2 ** (bits - 1)
    x_q = ((torch.round(x / (2.0 ** alpha * unit)) + zp).clamp(0, levels) - half).to(torch.int8)
    gamma = 1 + 0.5 * _normal(g, C)
    beta = 0.5 * _normal(g, C)
    # the output grid holds about six deviations on both sides
    return dict(x_q=x_q, zp_in=int(zp.item()) - half, alpha=alpha.to(torch.uint8), K=K,
                gamma=gamma, beta=beta, s_out=12.0 / levels, zp_out=0, bits=bits)


def _logits(g, G, Lq, Lk, s_logit):
    return torch.round(_normal(g, G, Lq, Lk) * (3.0 / s_logit)).to(torch.int32)


def _bias(g, Hb, Lq, Lk):
    if not Hb:
        return None
    return torch.randint(-64, 65, (Hb, Lq, Lk), generator=g, device=DEV, dtype=torch.int32)


def _qk_inputs(g, G, Lq, Lk, dk, zp, s_logit):
    """Q and K whose logits have a deviation of about 3 at scale s_logit (or as
    near as int8 allows)."""
    sigma = min(40.0, math.sqrt(3.0 / s_logit / math.sqrt(dk)))

    def one(L):
        return (torch.round(_normal(g, G, L, dk) * sigma) + zp).clamp(-128, 127).to(torch.int8)
    return one(Lq), one(Lk)


def _calls(case, g, prep):
    """The calls of one pass, in order, as functions of no arguments; each
    returns its outputs (None from a prepared call), and the buffers that
    prepared calls fill."""
    kind = case["kind"]
    out = []

    def empty(*shape, dtype):
        return torch.empty(shape, dtype=dtype, device=DEV) if prep else None

    def add(fn, *args, fills=None, **kw):
        if prep:
            out.append((fn(*args, prepare=True, **kw), fills))
        else:
            out.append((lambda: fn(*args, **kw), None))

    def add_ln(T, C, K, bits):
        p = _ln_inputs(g, T, C, K, bits)
        y = empty(T, C, dtype=torch.int8)
        add(fq.ptf_layernorm_int8, p["x_q"], p["zp_in"], p["alpha"], p["K"], p["gamma"], p["beta"],
            p["s_out"], p["zp_out"], p["bits"], y_q=y, fills=y)

    def add_qk(G, Lq, Lk, dk, d, bits, Hb, zp, s_logit):
        q, k = _qk_inputs(g, G, Lq, Lk, dk, zp, s_logit)
        v = _int8(g, -127, 127, G, Lk, d)
        o = empty(G, Lq, d, dtype=torch.int32)
        kw = dict(zp_q=zp, zp_k=-zp, bits=bits, bias=_bias(g, Hb, Lq, Lk))
        # V's scale over the LIS scale, against an output grid of about the
        # spread of an averaged V
        s_in, s_out = 2.0 ** -(2 ** bits - 1) / 127.0, 0.5 / 127.0
        if prep:
            y = empty(G, Lq, d, dtype=torch.int8)
            add(fq.lis_attention_qk, q, k, v, s_logit, out=o, fills=o, **kw)
            add(fq.requant_dyadic_int8, o, s_in, s_out, 0, y=y, fills=y)
            return

        def both():
            o = fq.lis_attention_qk(q, k, v, s_logit, **kw)
            return o, fq.requant_dyadic_int8(o, s_in, s_out, 0)
        out.append((both, None))

    if kind == "ln":
        add_ln(case["T"], case["C"], case["K"], case["bits"])
    elif kind == "head":
        G, Lq, Lk, d = case["G"], case["Lq"], case["Lk"], case["d"]
        logits = _logits(g, G, Lq, Lk, case["s_logit"])
        v = _int8(g, -127, 127, G, Lk, d)
        o = empty(G, Lq, d, dtype=torch.int32)
        add(fq.lis_attention_head, logits, v, case["s_logit"], bits=case["bits"],
            zp_v=case["zp_v"], bias=_bias(g, case["Hb"], Lq, Lk), out=o, fills=o)
    elif kind == "qk":
        add_qk(case["G"], case["Lq"], case["Lk"], case["dk"], case["d"], case["bits"], case["Hb"],
               case["zp"], case["s_logit"])
    elif kind == "maps":
        G, Lq, Lk, d, bits = case["G"], case["Lq"], case["Lk"], case["d"], case["bits"]
        logits = _logits(g, G, Lq, Lk, case["s_logit"])
        v = _int8(g, -127, 127, G, Lk, d)
        s, zp_v = case["s_logit"], case["zp_v"]
        product = fq.lis_attn_v_shift if bits <= 4 else fq.lis_attn_v_shift_wide
        if prep:
            codes = empty(G, Lq, fq.codes_ld(Lk, bits), dtype=torch.uint8)
            o = empty(G, Lq, d, dtype=torch.int32 if bits <= 4 else torch.int64)
            add(fq.lis_softmax_log4, logits, s, bits=bits, codes=codes, fills=codes)
            add(product, codes, v, Lk, zp_v=zp_v, bits=bits, out=o, fills=o)
        else:
            def both():
                codes = fq.lis_softmax_log4(logits, s, bits=bits)
                return codes, product(codes, v, Lk, zp_v=zp_v, bits=bits)
            out.append((both, None))
    elif kind == "calib":
        T, C, K, bits = case["T"], case["C"], case["K"], case["bits"]
        x = _activations(g, T, C)
        if prep:
            s, zp = empty(1, dtype=torch.float64), empty(1, dtype=torch.int32)
            alpha, x_q = empty(C, dtype=torch.uint8), empty(T, C, dtype=torch.int8)
            add(fq.ptf_calibrate, x, bits, K, s=s, zp=zp, alpha=alpha, fills=(s, zp, alpha))
            add(fq.ptf_quantize_int8, x, s, zp, alpha, bits, x_q=x_q, fills=x_q)
        else:
            def both():
                s, zp, alpha = fq.ptf_calibrate(x, bits, K)
                return (s, zp, alpha), fq.ptf_quantize_int8(x, s, zp, alpha, bits)
            out.append((both, None))
    else:
        add_ln(case["T"], case["C"], 3, 8)
        add_qk(case["G"], case["L"], case["L"], 64, case["d"], 4, 0, 0, S10)
    return out


def prepare(case, seed):
    return _calls(case, _gen(seed), bool(case["prepared"]))


def run(state):
    outputs = []
    for call, fills in state:
        got = call()
        outputs.append(got if fills is None else fills)
    return outputs


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how exact it is
# ---------------------------------------------------------------------------

def _attention(G, Lq, Lk, d, Hb=0, dk=0):
    """(bytes, flops) of attention with an int32 result: logits read, or Q and K."""
    n = G * Lq * Lk
    read = (G * (Lq + Lk) * dk if dk else 4 * n) + 4 * Hb * Lq * Lk + G * Lk * d
    return read + 4 * G * Lq * d, 2 * n * (d + dk) + 10 * n


def work(case):
    kind = case["kind"]
    if kind == "ln":
        n = case["T"] * case["C"]
        return {"bytes": 2 * n + 9 * case["C"], "flops": 12 * n}
    if kind == "calib":
        n = case["T"] * case["C"]
        # the grid depends on all of x, so x is read for the calibration and
        # again for the quantization; K + 1 candidate grids per element
        return {"bytes": 9 * n + 2 * case["C"], "flops": n * (8 * (case["K"] + 1) + 6)}
    if kind == "head":
        b, f = _attention(case["G"], case["Lq"], case["Lk"], case["d"], case["Hb"])
        return {"bytes": b, "flops": f}
    if kind == "maps":
        G, Lq, Lk, d, bits = case["G"], case["Lq"], case["Lk"], case["d"], case["bits"]
        b, f = _attention(G, Lq, Lk, d)
        codes = G * Lq * (Lk if bits > 4 else (Lk + 1) // 2)
        return {"bytes": b + 2 * codes + (4 * G * Lq * d if bits > 4 else 0), "flops": f}
    if kind == "qk":
        G, Lq, d = case["G"], case["Lq"], case["d"]
        b, f = _attention(G, Lq, case["Lk"], d, case["Hb"], case["dk"])
        return {"bytes": b + 5 * G * Lq * d, "flops": f + 4 * G * Lq * d}
    n = case["T"] * case["C"]
    b, f = _attention(case["G"], case["L"], case["L"], case["d"], 0, 64)
    out = case["G"] * case["L"] * case["d"]
    return {"bytes": 2 * n + 9 * case["C"] + b + 5 * out, "flops": 12 * n + f + 4 * out}


def tolerance(case):
    # Integer results of exact integer definitions, and a calibration whose
    # every operation is fixed (s is one correctly rounded binary64 expression).
    return "exact"


def exact(case, seed):
    """The scale of a calibration in plain torch; the integer outputs are
    compared exactly and need no reference in 64 bits."""
    if case["kind"] != "calib":
        return None
    x = _activations(_gen(seed), case["T"], case["C"])
    s = (x.max().double() - x.min().double()) / (2 ** case["bits"] - 1) / 2 ** case["K"]
    s = s.reshape(1)
    if case["prepared"]:
        return [(s, None, None), None]
    return [((s, None, None), None)]
