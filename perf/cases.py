"""The timed work of this framework: what a serving or evaluation program has it do.

Four kinds of call, each through the package's public entry points:

  prefill    hifa4_attention_fwd: the causal forward over whole prompts, fixed
             length (BSHD) or packed (THD with cu_seqlens), HIF4 operands with
             and without Smooth-QK, Q-Mean and the inconsistent normalizer, and
             the FP16-operand and P-only forms of the same loop;
  decode     hifa4_decode_fwd: one token per sequence over a packed HIF4 cache;
  cache      hifa4_quantize_qk and hifa4_quantize_v: writing that cache;
  calibrate  hifa4_calibrate_smooth_qk: the scales of one layer.

Shapes are the repository's own workloads (paper_2607_04302_amd/workloads.py)
and the lengths, head counts and raggedness its tests use.  Inputs follow the
same recipe as those workloads: Gaussian Q, K and V in fp16, with a few key
channels amplified as a QK-RMSNorm's affine weight does; the amplified channels
belong to the model and do not change with the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2607_04302_amd as h4

BLOCK = 64
PREFILL, DECODE, CACHE, CALIBRATE = "prefill", "decode", "cache", "calibrate"
OPERANDS = {"hif4": h4.OPERANDS_HIF4, "fp16": h4.OPERANDS_FP16, "p_only": h4.OPERANDS_P_ONLY}


def _prefill(name, batch, hq, hkv, d, s, lo=0, smooth=True, qmean=False, norm=0, operands="hif4", lens=0):
    """`lo` > 0: packed sequences of lengths drawn in [lo, s] from generator `lens`; else all of length s."""
    return {"name": name, "kind": PREFILL, "batch": batch, "hq": hq, "hkv": hkv, "d": d, "s": s, "lo": lo,
            "smooth": smooth, "qmean": qmean, "norm": norm, "operands": operands, "lens": lens}


def _decode(name, batch, hq, hkv, d, s, lo=0, smooth=True, norm=0, lens=0):
    return {"name": name, "kind": DECODE, "batch": batch, "hq": hq, "hkv": hkv, "d": d, "s": s, "lo": lo,
            "smooth": smooth, "norm": norm, "lens": lens}


def _cache(name, batch, hq, hkv, d, s, lo=0, smooth=True, with_q=False, lens=0):
    return {"name": name, "kind": CACHE, "batch": batch, "hq": hq, "hkv": hkv, "d": d, "s": s, "lo": lo,
            "smooth": smooth, "with_q": with_q, "lens": lens}


def _calibrate(name, n, hq, hkv, d, s, alpha=0.5):
    return {"name": name, "kind": CALIBRATE, "batch": n, "hq": hq, "hkv": hkv, "d": d, "s": s, "alpha": alpha}


def listed():
    return [
        # one short prompt, one head: the call's latency (the parity workload tiny_s256)
        _prefill("prefill_tiny_s256", 1, 1, 1, 128, 256),
        # one prompt of an 8B-class GQA layer: the headline workload
        _prefill("prefill_gqa_s4096", 1, 32, 8, 128, 4096),
        # a long prompt of the same layer: the largest work (long_s32768)
        _prefill("prefill_gqa_s32768", 1, 32, 8, 128, 32768),
        # a batch of packed prompts of mixed lengths, no smoothing (varlen_b16)
        _prefill("prefill_varlen_b16", 16, 32, 8, 128, 2048, lo=512, smooth=False),
        # wide heads, two prompts (wide_d256)
        _prefill("prefill_d256_s8192", 2, 16, 8, 256, 8192),
        # narrow heads without GQA, an odd length, with the Q-Mean auxiliary
        _prefill("prefill_d64_mha_qmean_s777", 3, 12, 12, 64, 777, qmean=True),
        # the same headline prompt on fp16 operands (the 16-bit form a user falls back to)
        _prefill("prefill_fp16_s4096", 1, 32, 8, 128, 4096, smooth=False, operands="fp16"),
        # one token for each of 8 long conversations (decode_b8_l32768)
        _decode("decode_b8_l32768", 8, 32, 8, 128, 32768),
        # one token of a single chat: the decode step's latency
        _decode("decode_b1_l4096", 1, 32, 8, 128, 4096),
        # a serving batch of conversations of mixed lengths
        _decode("decode_varlen_b32", 32, 32, 8, 128, 8192, lo=300),
        # writing the K^ and V^ cache of a prefilled batch
        _cache("cache_fill_b8_s4096", 8, 32, 8, 128, 4096),
        # the offline scales of one layer from 16 calibration prompts
        _calibrate("calibrate_n16_s4096", 16, 32, 8, 128, 4096),
    ]


# ---------------------------------------------------------------------------
# Drawn cases of the same ranges.
_MOST_FLOPS = 4.0 * 128 * 32 * (32768 * 32769 // 2)      # of prefill_gqa_s32768
_MOST_CACHE = 8 * 32768 * 8 * 128 * 2 * 36 // 64          # of decode_b8_l32768
_MOST_CALIB = 16 * 4096 * (32 + 8) * 128 * 2              # of calibrate_n16_s4096


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_heads(rng, groups):
    hkv = rng.choice([1, 2, 4, 8, 8, 12])
    return hkv * rng.choice(groups), hkv


def _draw_once(rng):
    kind = rng.choice([PREFILL] * 10 + [DECODE] * 5 + [CACHE] * 3 + [CALIBRATE] * 2)
    d = rng.choice([64, 128, 128, 128, 256])
    smooth = rng.random() < 0.7
    lens = rng.randrange(1, 1 << 20)
    if kind == PREFILL:
        hq, hkv = _draw_heads(rng, [1, 2, 3, 4, 4, 5, 8])
        s = _log_int(rng, 16, 32768)
        batch = _log_int(rng, 1, 16)
        lo = max(1, s // rng.randrange(2, 9)) if batch > 1 and rng.random() < 0.5 else 0
        operands = rng.choice(["hif4"] * 7 + ["fp16"] * 2 + ["p_only"])
        hif4 = operands == "hif4"
        return _prefill("", batch, hq, hkv, d, s, lo, smooth and hif4, hif4 and rng.random() < 0.15,
                        1 if operands != "fp16" and rng.random() < 0.2 else 0, operands, lens)
    if kind == DECODE:
        hq, hkv = _draw_heads(rng, [1, 2, 3, 4, 4, 5, 8])
        s = _log_int(rng, 64, 32768)
        batch = _log_int(rng, 1, 64)
        lo = max(1, s // rng.randrange(2, 17)) if batch > 1 and rng.random() < 0.6 else 0
        return _decode("", batch, hq, hkv, d, s, lo, smooth, 1 if rng.random() < 0.2 else 0, lens)
    if kind == CACHE:
        hq, hkv = _draw_heads(rng, [1, 2, 4, 8])
        s = _log_int(rng, 1, 32768)
        batch = _log_int(rng, 1, 32)
        lo = max(1, s // rng.randrange(2, 9)) if batch > 1 and rng.random() < 0.5 else 0
        return _cache("", batch, hq, hkv, d, s, lo, smooth, rng.random() < 0.3, lens)
    hq, hkv = _draw_heads(rng, [1, 2, 4, 8])
    return _calibrate("", _log_int(rng, 1, 16), hq, hkv, d, _log_int(rng, 100, 8192), rng.choice([-1.0, 0.25, 0.5]))


def _fits(c):
    kv = _tokens(c) * c["hkv"] * c["d"]
    if c["kind"] == PREFILL:
        return work(c)["flops"] <= _MOST_FLOPS and c["batch"] * c["s"] <= 32768 and kv <= 1 << 26
    if c["kind"] == DECODE:
        return c["batch"] * c["s"] * c["hkv"] * c["d"] * 2 * 36 // 64 <= _MOST_CACHE
    if c["kind"] == CACHE:
        return c["batch"] * c["s"] * c["d"] * (c["hq"] + 2 * c["hkv"]) <= 1 << 28
    return _tokens(c) * (c["hq"] + c["hkv"]) * c["d"] * 2 <= _MOST_CALIB


def draw(rng):
    while True:
        c = _draw_once(rng)
        if _fits(c):
            del c["name"]
            return c


# ---------------------------------------------------------------------------
# Inputs.
def _lengths(c):
    if c.get("lo", 0) <= 0:
        return [c["s"]] * c["batch"]
    g = np.random.default_rng(c["lens"])
    return [int(x) for x in g.integers(c["lo"], c["s"] + 1, c["batch"])]


def _packed(c):
    return c.get("lo", 0) > 0


def _tokens(c):
    return sum(_lengths(c))


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed, dev):
    return torch.Generator(device=dev).manual_seed(int(seed) & 0x7FFFFFFFFFFF)


def _gain(c, dev):
    """[Hkv, D] factors of the key channels: the model's amplified channels (x16), ones elsewhere."""
    g = np.random.default_rng(4242)
    gain = np.ones((c["hkv"], c["d"]), np.float32)
    for h in range(c["hkv"]):
        gain[h, g.choice(c["d"], c["d"] // 32, replace=False)] = 16.0
    return torch.from_numpy(gain).to(dev)


def _normal(shape, gen, dev):
    return torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)


def _draws(c, seed):
    """q, k, v (fp16) of the case: prefill and cache [T, H, D], decode q [B, Hq, D], calibrate [n*S, H, D]."""
    dev = _device()
    gen = _gen(seed, dev)
    t = _tokens(c)
    nq = c["batch"] if c["kind"] == DECODE else t
    q = _normal((nq, c["hq"], c["d"]), gen, dev).half()
    k = _normal((t, c["hkv"], c["d"]), gen, dev)
    k = (k * _gain(c, dev)).half() if c.get("smooth", True) else k.half()
    v = _normal((t, c["hkv"], c["d"]), gen, dev).half() if c["kind"] != CALIBRATE else None
    return q, k, v


def _scales(c, dev):
    """Smooth-QK scales [Hkv, D] of the model (Eq. 1 with alpha 1/2), from one prompt that no seed changes."""
    if not c["smooth"]:
        return None
    gen = _gen(77, dev)
    q = _normal((512, c["hkv"], c["hq"] // c["hkv"], c["d"]), gen, dev).half().abs().amax((0, 2)).double()
    k = (_normal((512, c["hkv"], c["d"]), gen, dev) * _gain(c, dev)).half().abs().amax(0).double()
    return (k / q).sqrt().float()


def _cu(c, dev):
    return torch.tensor([0] + list(np.cumsum(_lengths(c))), dtype=torch.int32, device=dev)


def _laid_out(c, x):
    """[T, H, D] as the entry points take it: packed, or [B, S, H, D]."""
    return x if _packed(c) else x.view(c["batch"], c["s"], x.shape[1], x.shape[2])


def prepare(case, seed):
    c = case
    q, k, v = _draws(c, seed)
    dev = q.device
    seqs = {"cu_seqlens": _cu(c, dev), "max_seqlen": c["s"]} if _packed(c) else {}
    st = {"case": c, "seqs": seqs}
    if c["kind"] == PREFILL:
        st.update(q=_laid_out(c, q), k=_laid_out(c, k), v=_laid_out(c, v), s=_scales(c, dev))
    elif c["kind"] == DECODE:
        s = _scales(c, dev)
        _, _, kc, km = h4.hifa4_quantize_qk(None, _laid_out(c, k), s, **seqs)
        vc, vm = h4.hifa4_quantize_v(_laid_out(c, v), **seqs)
        st.update(q=q, kc=kc, km=km, vc=vc, vm=vm, s=s)
    elif c["kind"] == CACHE:
        st.update(q=_laid_out(c, q) if c["with_q"] else None, k=_laid_out(c, k), v=_laid_out(c, v), s=_scales(c, dev))
    else:
        st.update(q=q.view(c["batch"], c["s"], c["hq"], c["d"]), k=k.view(c["batch"], c["s"], c["hkv"], c["d"]))
    return st


def run(state):
    c, x = state["case"], state
    if c["kind"] == PREFILL:
        o, lse = h4.hifa4_attention_fwd(x["q"], x["k"], x["v"], x["s"], norm=c["norm"], operands=OPERANDS[c["operands"]],
                                        q_mean=c["qmean"], **x["seqs"])
        return {"o": o, "lse": lse}
    if c["kind"] == DECODE:
        o, lse = h4.hifa4_decode_fwd(x["q"], x["kc"], x["km"], x["vc"], x["vm"], x["s"], norm=c["norm"], **x["seqs"])
        return {"o": o, "lse": lse}
    if c["kind"] == CACHE:
        qc, qm, kc, km = h4.hifa4_quantize_qk(x["q"], x["k"], x["s"], **x["seqs"])
        vc, vm = h4.hifa4_quantize_v(x["v"], **x["seqs"])
        out = {"k_codes": kc, "k_meta": km, "v_codes": vc, "v_meta": vm}
        if qc is not None:
            out.update(q_codes=qc, q_meta=qm)
        return out
    s, rep = h4.hifa4_calibrate_smooth_qk(x["q"], x["k"], c["alpha"])
    return {"s": s, "rho_k": rep["rho_k"], "t_kq": rep["t_kq"], "branch": rep["branch"], "alpha_used": rep["alpha_used"]}


# ---------------------------------------------------------------------------
def work(case):
    c = case
    lens = _lengths(c)
    t, d, hq, hkv = sum(lens), c["d"], c["hq"], c["hkv"]
    scales = 4 * hkv * d if c.get("smooth") else 0
    packed_k = t * hkv * (d // 64) * 36
    if c["kind"] == PREFILL:
        pairs = sum(n * (n + 1) // 2 for n in lens)
        return {"bytes": t * d * 2 * (2 * hq + 2 * hkv) + 4 * hq * t + scales, "flops": 4.0 * d * hq * pairs}
    if c["kind"] == DECODE:
        blocks = sum((n + 63) // 64 for n in lens)
        return {"bytes": packed_k + blocks * hkv * d * 36 + c["batch"] * hq * (4 * d + 4) + scales,
                "flops": 4.0 * d * hq * t}
    if c["kind"] == CACHE:
        groups = c["batch"] * ((c["s"] + 63) // 64) * hkv * d
        n = t * d * 2 * 2 * hkv + packed_k + groups * 36 + scales
        if c["with_q"]:
            n += t * hq * (2 * d + d // 64 * 36)
        return {"bytes": n, "flops": 0}
    return {"bytes": t * d * 2 * (hq + hkv) + 4 * hkv * d, "flops": 0}


def tolerance(case):
    """Prefill: every score, weight and code of the HIF4 form is fixed by the contract; the fp32 sums of O and l and
    the rounding of O to fp16 are free (2e-4 from the 64-bit result on every listed case, FP16 operands included,
    whose scores are fp32 sums in a free order).  Decode: besides, the scaled score may reach fp16 in one rounding or
    in two, which moves one score in some thousands to its neighbour, by up to 2^-7: a key that dominates its row
    then moves the row by half a percent (4e-4 seen over 1024 rows; a call may have a few rows only).  Codes are
    whole numbers and stay the same; the scales of a calibration are float64 rounded once to fp32 (2e-8 seen)."""
    return {CACHE: "exact", CALIBRATE: {"rel": 1e-7}, DECODE: {"rel": 3e-3}, PREFILL: {"rel": 1e-3}}[case["kind"]]


# ---------------------------------------------------------------------------
# The same results in 64 bits from plain torch: the roundings the contract
# states (fp16 operands, scores and weights, HIF4 codes) are kept, every free
# sum and quotient is float64.
_TABLES = {}


def _table(name, dev):
    if (name, str(dev)) not in _TABLES:
        if name == "exp2":             # fp16(2^x) for every fp16 x, rounded once
            x = np.arange(65536, dtype=np.uint16).view(np.float16).astype(np.float64)
            with np.errstate(all="ignore"):
                t = np.exp2(x).astype(np.float16).astype(np.float64)
        else:                          # the 256 E6M2 values, ascending
            b = np.arange(256)
            t = (1.0 + (b & 3) / 4.0) * np.exp2((b >> 2) - 31.0)
        _TABLES[name, str(dev)] = torch.from_numpy(t).to(dev)
    return _TABLES[name, str(dev)]


def _rn16(x):
    """float64 to fp16, rounded once (through a round-to-odd float32)."""
    f = x.float()
    fd = f.double()
    b = f.view(torch.int32)
    b = torch.where(fd.abs() > x.abs(), b - 1, b)
    b = torch.where(fd != x, b | 1, b)
    return b.view(torch.float32).half()


def _exp2_16(x16):
    return _table("exp2", x16.device)[(x16.view(torch.int16).int() & 0xFFFF).long()]


def _hif4(x):
    """HIF4 of groups of 64 along the last axis (float64): (values / (b/4), b, codes, metadata words)."""
    e6m2 = _table("e6m2", x.device)
    a = x.abs()
    a8 = a.view(*a.shape[:-1], 8, 8).amax(-1)
    a4 = a.view(*a.shape[:-1], 16, 4).amax(-1)
    base = torch.searchsorted(1.75 * e6m2, a8.amax(-1))
    b = e6m2[base]
    e2 = a8 <= 0.875 * b[..., None]
    e3 = a4 <= 0.875 * b[..., None] * torch.where(e2, 0.5, 1.0).repeat_interleave(2, -1)
    sh = e2.repeat_interleave(2, -1).double() + e3.double()
    unit = torch.exp2(-sh).repeat_interleave(4, -1)
    u = torch.floor(a / (unit * (b[..., None] / 4)) + 0.5)
    o = torch.where(x < 0, -u, u) * unit
    return o, b, u, (base, e2, e3)


def _codes(x, o, u, meta):
    base, e2, e3 = meta
    nib = (u.int() | ((o < 0).int() << 3))
    by = (nib[..., 0::2] | (nib[..., 1::2] << 4)).to(torch.uint8)
    w = base.long()
    for j in range(8):
        w = w | (e2[..., j].long() << (8 + j))
    for j in range(16):
        w = w | (e3[..., j].long() << (16 + j))
    w = torch.where(w >= 1 << 31, w - (1 << 32), w)
    return by, w.int()


def _smoothed(c, q, k, dev):
    s = _scales(c, dev)
    if s is None or c.get("operands", "hif4") != "hif4":
        return q, k
    sq = s.double().repeat_interleave(c["hq"] // c["hkv"], 0)
    return _rn16(q.double() * sq), _rn16(k.double() / s.double())


def _v_groups(v, n):
    """[L, H, D] -> [NB, H, D, 64] float64, zero padded."""
    nb = (n + BLOCK - 1) // BLOCK
    x = torch.zeros((nb * BLOCK,) + tuple(v.shape[1:]), dtype=torch.float64, device=v.device)
    x[:n] = v[:n].double()
    return x.view(nb, BLOCK, v.shape[1], v.shape[2]).permute(0, 2, 3, 1).contiguous()


def _attend(c, q, k, v, rows):
    """Algorithm 1's loop for query rows `rows` (ascending positions, all heads) of one sequence: q [R, Hq, D]
    (smoothed), k, v [L, Hkv, D].  Returns o [R, Hq, D] and lse [Hq, R] in float64."""
    dev, d, hq, hkv, n = q.device, c["d"], c["hq"], c["hkv"], k.shape[0]
    grp, g = hq // hkv, c["d"] // 64
    operands = c.get("operands", "hif4")
    qt = q.double().permute(1, 0, 2).contiguous()                              # [Hq, R, D]
    kt = k.double().permute(1, 0, 2).contiguous()
    nr = qt.shape[1]
    mu = kappa = None
    if operands == "hif4":
        if c.get("qmean"):
            mu = _rn16(qt.sum(-1) / d)
            kappa = kt.sum(-1).float()
            qt = (qt.half() - mu[..., None]).double()
            mu = mu.double()
        o, b, _, _ = _hif4(qt.view(hq, nr, g, 64))
        qt = (o * (b[..., None] / 4)).view(hq, nr, d)
        o, b, _, _ = _hif4(kt.view(hkv, n, g, 64))
        kt = (o * (b[..., None] / 4)).view(hkv, n, d)
        o, b, _, _ = _hif4(_v_groups(v, n))
        vt = (o * (b[..., None] / 4)).permute(1, 0, 3, 2).contiguous()          # [Hkv, NB, 64, D]
    else:
        vt = _v_groups(v, n).permute(1, 0, 3, 2).contiguous()
    scale = torch.tensor(math.log2(math.e) / math.sqrt(d), dtype=torch.float32, device=dev)
    inf16 = torch.tensor(-math.inf, dtype=torch.float16, device=dev)
    pos = torch.as_tensor(rows, device=dev)
    m = torch.full((hq, nr), -math.inf, dtype=torch.float16, device=dev)
    out = torch.zeros((hq, nr, d), dtype=torch.float64, device=dev)
    l = torch.zeros((hq, nr), dtype=torch.float64, device=dev)
    for j in range((n + BLOCK - 1) // BLOCK):
        r0 = int((pos < BLOCK * j).sum()) if nr > 1 else 0
        keys = kt[:, BLOCK * j:BLOCK * j + BLOCK]
        nk = keys.shape[1]
        a = qt[:, r0:].reshape(hkv, grp * (nr - r0), d)
        if operands == "hif4":
            acc = None
            for i in range(g):
                t = torch.bmm(a[..., 64 * i:64 * i + 64].contiguous(),
                              keys[..., 64 * i:64 * i + 64].transpose(1, 2).contiguous()).float()
                acc = t if acc is None else acc + t
            acc = acc.view(hq, nr - r0, nk)
            if mu is not None:
                kap = kappa[:, BLOCK * j:BLOCK * j + nk].double().repeat_interleave(grp, 0)
                acc = (acc.double() + mu[:, r0:, None] * kap[:, None, :]).float()
        else:
            acc = torch.bmm(a, keys.transpose(1, 2).contiguous()).float().view(hq, nr - r0, nk)
        s2 = (acc * scale).half()
        hidden = (BLOCK * j + torch.arange(nk, device=dev))[None, :] > pos[r0:, None]
        s2 = torch.where(hidden, inf16, s2)
        m_old = m[:, r0:]
        m_new = torch.maximum(m_old, s2.amax(-1))
        r = _exp2_16(m_old - m_new)
        p = torch.zeros((hq, nr - r0, BLOCK), dtype=torch.float64, device=dev)
        p[..., :nk] = _exp2_16(s2 - m_new[..., None])
        ph = p
        if operands != "fp16":
            o, b, _, _ = _hif4(p)
            ph = o * (b[..., None] / 4)
        pv = torch.bmm(ph.reshape(hkv, grp * (nr - r0), BLOCK), vt[:, j].contiguous()).view(hq, nr - r0, d)
        out[:, r0:] = out[:, r0:] * r[..., None] + pv
        l[:, r0:] = l[:, r0:] * r + (p if c.get("norm", 0) == 1 else ph).sum(-1)
        m[:, r0:] = m_new
    return (out / l[..., None]).permute(1, 0, 2), m.double() * math.log(2.0) + torch.log(l)


def _exact_attention(c, seed):
    q, k, v = _draws(c, seed)
    dev = q.device
    if c["kind"] == PREFILL and work(c)["flops"] > 1.01 * _MOST_FLOPS:
        return None
    q, k = _smoothed(c, q, k, dev)
    lens = _lengths(c)
    dec = c["kind"] == DECODE
    o = torch.zeros(q.shape, dtype=torch.float64, device=dev)
    lse = torch.zeros((c["hq"], q.shape[0]), dtype=torch.float64, device=dev)
    t0 = 0
    for b, n in enumerate(lens):
        at = slice(b, b + 1) if dec else slice(t0, t0 + n)
        o[at], lse[:, at] = _attend(c, q[at], k[t0:t0 + n], v[t0:t0 + n], [n - 1] if dec else list(range(n)))
        t0 += n
    return {"o": o if dec else _laid_out(c, o), "lse": lse}


def _exact_cache(c, seed):
    q, k, v = _draws(c, seed)
    qs, ks = _smoothed(c, q, k, q.device)
    g = c["d"] // 64

    def rows(x):
        by, w = [], []
        for part in x.double().split(8192):
            y = part.view(part.shape[0], part.shape[1], g, 64)
            o, _, u, meta = _hif4(y)
            cc, ww = _codes(y, o, u, meta)
            by.append(cc)
            w.append(ww)
        return torch.cat(by), torch.cat(w)

    out = {}
    out["k_codes"], out["k_meta"] = rows(ks)
    if c["with_q"]:
        out["q_codes"], out["q_meta"] = rows(qs)
    nb = (c["s"] + BLOCK - 1) // BLOCK
    vc = torch.zeros((c["batch"], nb, c["hkv"], c["d"], 32), dtype=torch.uint8, device=q.device)
    vm = torch.zeros((c["batch"], nb, c["hkv"], c["d"]), dtype=torch.int32, device=q.device)
    t0 = 0
    for b, n in enumerate(_lengths(c)):
        y = _v_groups(v[t0:t0 + n], n)
        o, _, u, meta = _hif4(y)
        vc[b, :y.shape[0]], vm[b, :y.shape[0]] = _codes(y, o, u, meta)
        t0 += n
    out["v_codes"], out["v_meta"] = vc, vm
    return out


def _exact_calibrate(c, seed):
    q, k, _ = _draws(c, seed)
    n, hkv, d = c["batch"], c["hkv"], c["d"]
    qm = q.view(n, c["s"], hkv, c["hq"] // hkv, d).abs().amax((1, 3)).double()
    km = k.view(n, c["s"], hkv, d).abs().amax(1).double()
    qb, kb = qm.square().mean(0).sqrt(), km.square().mean(0).sqrt()
    bits = (k.view(torch.int16).int() & 0x7FFF).view(-1)
    hist = torch.zeros(32768, dtype=torch.float64, device=k.device)
    for part in bits.split(1 << 24):
        hist += torch.bincount(part, minlength=32768)
    cum = torch.cumsum(hist, 0)
    total = int(cum[-1])
    at = 0.99 * (total - 1)
    lo = int(math.floor(at))

    def order(i):
        b = int(torch.searchsorted(cum, torch.tensor([float(i)], dtype=torch.float64, device=k.device), right=True))
        return float(np.array([b], dtype=np.uint16).view(np.float16)[0])

    x, y = order(lo), order(min(lo + 1, total - 1))
    p99 = x + (y - x) * (at - lo)
    rho, t_kq = float(km.max()) / p99, float(km.max()) / float(qm.max())
    alpha = c["alpha"]
    if alpha < 0:
        branch = 0 if rho < 6 or t_kq < 2 else 2 if t_kq > 3 else 1
        alpha = {0: 0.0, 1: 0.25, 2: 0.5}[branch]
    else:
        branch = 0 if alpha == 0 else 2 if alpha >= 0.5 else 1
    s = kb.pow(alpha) / qb.pow(1.0 - alpha) if alpha else torch.ones_like(kb)
    return {"s": s, "rho_k": rho, "t_kq": t_kq, "branch": branch, "alpha_used": alpha}


def exact(case, seed):
    if case["kind"] in (PREFILL, DECODE):
        return _exact_attention(case, seed)
    if case["kind"] == CACHE:
        return _exact_cache(case, seed)
    return _exact_calibrate(case, seed)
