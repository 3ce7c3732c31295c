"""Performance cases of the 3-bit KV-cache path: what a program that serves a RoPE transformer with this
library has it do, through its public entry points.

A case is a dict of plain values; its "op" names the entry point:
  decode_step     append one token per sequence and attend over the cache
  decode_attend   attend over the cache (the second of the two calls of a step)
  quantize        prefill, or append a few tokens to sequences that are cached already
  quantize_ragged prefill of sequences of different lengths in one call
  dequantize      fp16 key and value rows of every cached token
  calibrate_rotation, calibrate_tables   once per model and layer: Pi per head; the K and V tables and the
                  mean residuals per head
Sizes are those of the repository's workloads (20 heads x 33 layers, 40 heads x 36 layers, 1024 and 8192
tokens, 64 ragged sequences, 4096 calibration vectors per head) and what lies around them.

Inputs are drawn here from a seed, and a decode case's cache is quantized here in plain torch, so that a
decode case does not depend on the library's own quantizer. exact() evaluates a case in 64 bits in torch.
"""
import math

import torch

import paper_2603_26110_amd as tq

D = 64
ALPHA = math.sqrt(math.pi / 2) / D
GAUSS8 = (-2.152, -1.344, -0.7560, -0.2451, 0.2451, 0.7560, 1.344, 2.152)
DEV = "cuda"

_BASE = {"layers": 1, "heads": 20, "batch": 1, "tokens": 1024, "shortest": 0, "cached": 0, "half_precision": True,
         "v_rotate": True, "v_signs": False, "per_element": False, "rope_half": False, "fp32_out": False}


def _case(op, name=None, **kw):
    c = dict(_BASE, op=op, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # One sequence's next token in one layer: the call a model's attention layer makes per generated token.
        _case("decode_step", "step_layer"),
        # The same for all 33 layers in one launch: the benchmark's step.
        _case("decode_step", "step_model", layers=33),
        # One layer of a batch of 64 sequences of 50 to 1024 cached tokens (a serving batch).
        _case("decode_step", "step_ragged_layer", batch=64, shortest=50),
        # One layer of 16 sequences of 8192 cached tokens, 40 heads: the longest contexts, bound by memory.
        _case("decode_step", "step_long_layer", heads=40, batch=16, tokens=8192),
        # The paper's residual form on K and V, fp32 in and out, an odd length, the other RoPE pairing.
        _case("decode_attend", "attend_per_element", batch=8, tokens=777, half_precision=False, v_signs=True,
              per_element=True, rope_half=True),
        # Prefill of one sequence in one layer (a model prefills layer by layer).
        _case("quantize", "prefill_layer"),
        # Prefill of the whole 33-layer cache in one call: the benchmark's prefill.
        _case("quantize", "prefill_model", layers=33),
        # Prefill of a ragged batch of 64 sequences in one layer.
        _case("quantize_ragged", "prefill_ragged_layer", batch=64, shortest=50),
        # One token appended to each of 64 cached sequences in one layer (a step as two calls).
        _case("quantize", "append_batch", batch=64, tokens=1, cached=300),
        # fp16 rows of the whole 33-layer cache (dequantize, then attend elsewhere).
        _case("dequantize", "dequantize_model", layers=33),
        # Calibration of one layer: Pi of each head from 4096 post-RoPE keys.
        _case("calibrate_rotation", "calibrate_rotation_layer", tokens=4096),
        # Calibration of one layer: K and V tables and mean residuals from 4096 vectors per head.
        _case("calibrate_tables", "calibrate_tables_layer", tokens=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode_step", "decode_step", "decode_attend", "quantize", "quantize", "quantize_ragged",
                     "dequantize", "calibrate_rotation", "calibrate_tables"])
    kw = {"heads": rng.choice([1, 5, 12, 20, 33, 40]), "rope_half": rng.random() < 0.2}
    if op.startswith("calibrate"):
        return _case(op, heads=rng.randint(1, 40) if op == "calibrate_rotation" else rng.randint(1, 20),
                     tokens=_log(rng, 200, 4096), v_rotate=rng.random() < 0.75)
    kw["half_precision"] = rng.random() < 0.75
    kw["v_rotate"] = rng.random() < 0.8
    kw["v_signs"] = rng.random() < 0.25
    kw["per_element"] = rng.random() < 0.25
    kw["fp32_out"] = rng.random() < 0.2
    most = 5_000_000 if op.startswith("decode") else 660_000       # token-heads
    kw["tokens"] = _log(rng, 1, 8192)
    if op == "quantize_ragged":
        kw["tokens"] = max(2, kw["tokens"])
    if op == "quantize" and rng.random() < 0.5:
        kw["tokens"] = _log(rng, 1, 63)
    if op == "quantize":
        kw["cached"] = rng.choice([0, rng.randint(1, 500)])
    room = max(1, most // (kw["heads"] * kw["tokens"]))
    kw["batch"] = _log(rng, 1, max(1, min(64, room)))
    kw["layers"] = rng.choice([1, 1, max(1, min(36, room // kw["batch"]))])
    if op == "quantize_ragged" or (op != "quantize" and kw["tokens"] > 1 and rng.random() < 0.5):
        kw["shortest"] = rng.randint(1, max(1, kw["tokens"] - 1))
    return _case(op, **kw)


# ------------------------------------------------------------------ inputs
def _flags(case):
    f = tq.V_ROTATE if case["v_rotate"] else 0
    for key, bit in (("v_signs", tq.V_QJL), ("per_element", tq.QJL_PAPER), ("rope_half", tq.ROPE_HALF),
                     ("fp32_out", tq.OUT_FP32)):
        f |= bit if case[key] else 0
    return f


def _lengths(case, seed):
    """Tokens of each sequence and its first slot; the slots in all. A ragged batch's lengths belong to the case
    (uniform, the longest case["tokens"]), their order to the seed, so that every seed has the same sizes."""
    B, T = case["batch"], case["tokens"]
    lens = torch.full((B,), T, dtype=torch.int64)
    if case["shortest"]:
        lens = torch.randint(case["shortest"], T + 1, (B,), generator=torch.Generator().manual_seed(B * 10007 + T))
        lens[B - 1] = T
        lens = lens[torch.randperm(B, generator=torch.Generator().manual_seed(seed * 7 + 1))]
    caps = (lens + case["cached"] + 1 + 63) // 64 * 64
    first = torch.cumsum(caps, 0) - caps
    return lens, first, int(caps.sum())


def _generator(seed, *more):
    s = seed
    for m in more:
        s = s * 1000003 + m + 1
    return torch.Generator(device=DEV).manual_seed(s % (1 << 62))


def _randn(g, *shape, dtype=torch.float32):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype)


def _parameters(case, seed):
    """Pi (random rotations), S, the K and V tables and the mean residuals, as calibration leaves them."""
    L, H = case["layers"], case["heads"]
    g = _generator(seed, 1)
    pi = torch.eye(D, device=DEV, dtype=torch.float64).expand(L, H, D, D).contiguous()
    for _ in range(D):                                             # products of reflections
        w = _randn(g, L, H, D, 1, dtype=torch.float64)
        w /= w.norm(dim=2, keepdim=True)
        pi -= 2 * w * (w * pi).sum(2, keepdim=True)
    base = torch.tensor(GAUSS8, device=DEV)
    lut = [(base + 0.02 * _randn(g, L, H, 8)).contiguous() for _ in range(2)]
    ebar = 0.15 * (1 + 0.05 * _randn(g, L, H, 2))
    return {"pi": pi.float().contiguous(), "S": _randn(g, D, D), "lut_k": lut[0], "lut_v": lut[1], "ebar": ebar}


def _outliers(case, seed):
    """[L][1][H][64] key scale: four outlier channels per head, 20 times the others."""
    g = _generator(seed, 2)
    L, H = case["layers"], case["heads"]
    at = torch.rand((L, H, D), generator=g, device=DEV).argsort(-1)[..., :4]
    return torch.ones((L, H, D), device=DEV).scatter_(2, at, 20.0)[:, None]


def _kv(case, g, scale, n):
    """Raw keys and values [L][n][H][64]: Gaussian keys with outlier channels, Student-t values (4 degrees)."""
    shape = (case["layers"], n, case["heads"], D)
    k = _randn(g, *shape) * scale
    chi = sum(_randn(g, *shape).square_() for _ in range(4))
    v = _randn(g, *shape) / torch.sqrt(chi / 4)
    return (k.half(), v.half()) if case["half_precision"] else (k, v)


# ------------------------------------------------- the method in plain torch
def _rope(x, pos, half):
    """x [..., n, H, 64] at positions pos [n], in x's precision (angles in 64 bits)."""
    m = torch.arange(D // 2, device=DEV, dtype=torch.float64)
    a = pos.to(DEV, torch.float64)[:, None] * torch.pow(10000.0, -2 * m / D)
    c, s = a.cos().to(x.dtype)[:, None, :], a.sin().to(x.dtype)[:, None, :]
    y = torch.empty_like(x)
    lo, hi = (slice(0, 32), slice(32, 64)) if half else (slice(0, 64, 2), slice(1, 64, 2))
    p, q = x[..., lo], x[..., hi]
    y[..., lo], y[..., hi] = p * c - q * s, p * s + q * c
    return y


def _rotate(x, pi):
    """x [L][n][H][64] -> Pi x per head (pi [L][H][64][64])."""
    return torch.matmul(x.transpose(1, 2), pi.to(x.dtype).transpose(-1, -2).contiguous()).transpose(1, 2)


def _quantize(x, lut, S, signs):
    """Indices, sign bits, norm and residual norm of x^ [L][n][H][64]; signs: "none", "projected" or "element"."""
    c = lut.to(x.dtype)
    t = (0.5 * (lut[..., 1:] + lut[..., :-1])).to(x.dtype)
    n = x.norm(dim=-1, keepdim=True)
    u = torch.where(n > 0, x * (8.0 / n), torch.zeros_like(x))
    idx = torch.zeros(u.shape, dtype=torch.int64, device=DEV)
    for m in range(7):
        idx += u > t[:, None, :, m:m + 1]
    r = u - torch.gather(c[:, None].expand(*u.shape[:-1], 8), -1, idx)
    g = r.norm(dim=-1, keepdim=True)
    bit = torch.zeros_like(idx)
    if signs == "projected":
        bit = (~(r @ S.to(x.dtype).T.contiguous() < 0)).long()
    elif signs == "element":
        bit = (~(r < 0)).long()
    return idx, bit, n[..., 0], torch.zeros_like(g[..., 0]) if signs == "none" else g[..., 0]


def _quantize_kv(case, par, k, v, pos):
    signs = "element" if case["per_element"] else "projected"
    kq = _quantize(_rotate(_rope(k, pos, case["rope_half"]), par["pi"]), par["lut_k"], par["S"], signs)
    vx = _rotate(v, par["pi"]) if case["v_rotate"] else v
    return kq, _quantize(vx, par["lut_v"], par["S"], signs if case["v_signs"] else "none")


def _int32(w):
    return torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)


def _pack_sequence(planes, first, kq, vq):
    """Writes a sequence's codes into the planes (views by _planes) at its first slot, a multiple of 64."""
    n = kq[0].shape[1]
    full = (n + 63) // 64 * 64
    j = torch.arange(8, device=DEV)
    kb = (kq[0].unflatten(-1, (8, 8)) << (3 * j)).sum(-1) | (kq[1].unflatten(-1, (8, 8)) << (24 + j)).sum(-1)
    nib = torch.nn.functional.pad(vq[0] | (vq[1] << 3), (0, 0, 0, 0, 0, full - n))     # [L][full][H][64]
    kb = torch.nn.functional.pad(kb, (0, 0, 0, 0, 0, full - n))
    k = kb.transpose(1, 2).unflatten(2, (full // 64, 64)).unflatten(-1, (2, 4)).transpose(3, 4)
    v = nib.transpose(1, 2).unflatten(2, (full // 64, 2, 4, 8))
    v = (v << (4 * j)[:, None]).sum(5).transpose(4, 5)                                # [L][H][tile][2][64][4]
    at = first // 64
    planes[0][:, :, at:at + full // 64] = _int32(k)
    planes[1][:, :, at:at + full // 64] = _int32(v)
    sc = torch.stack([kq[2], kq[3], vq[2], vq[3]], -1).transpose(1, 2)
    planes[2][:, :, first:first + n] = sc.clamp(max=65504.0).half()


def _planes(case, cache, slots):
    """K [L][H][tile][2][slot][4 words], V [L][H][tile][2][dim][4 words], scalars [L][H][slot][4] views."""
    L, H = case["layers"], case["heads"]
    k, v, s = cache
    return (k.view(torch.int32).view(L, H, slots // 64, 2, 64, 4), v.view(torch.int32).view(L, H, slots // 64, 2, 64, 4),
            s.view(torch.float16).view(L, H, slots, 4))


def _fill(case, par, scale, seed, cache, first, lens, slots):
    """Quantizes the cached tokens of every sequence into the cache."""
    planes = _planes(case, cache, slots)
    for b, n in enumerate(lens.tolist()):
        if n:
            k, v = _kv(case, _generator(seed, 3, b), scale, n)
            _pack_sequence(planes, int(first[b]), *_quantize_kv(case, par, k.float(), v.float(), torch.arange(n)))


def _unpack(planes, l, first, n):
    """fp64 indices and +-1 signs of a sequence's keys and values in layer l: four [H][n][64], and scalars [H][n][4]."""
    full, at = (n + 63) // 64 * 64, first // 64
    j = torch.arange(8, device=DEV, dtype=torch.int32)
    k = planes[0][l, :, at:at + full // 64].transpose(2, 3).flatten(3, 4)              # [H][tile][slot][8 words]
    ki = ((k[..., None] >> (3 * j)) & 7).flatten(3, 4).flatten(1, 2)[:, :n].long()
    ks = ((k[..., None] >> (24 + j)) & 1).flatten(3, 4).flatten(1, 2)[:, :n].double() * 2 - 1
    v = planes[1][l, :, at:at + full // 64]                                            # [H][tile][2][dim][4]
    v = ((v[..., None] >> (4 * j)) & 15).movedim(3, 5).flatten(1, 4)[:, :n]            # [H][tokens][dim]
    return ki, ks, (v & 7).long(), (v >> 3).double() * 2 - 1, planes[2][l, :, first:first + n].double()


def _rows(case, par, l, codes):
    """k~ and v~ [H][n][64] of the unpacked codes, in 64 bits."""
    ki, ks, vi, vs, sc = codes
    S, ebar = par["S"].double(), par["ebar"][l].double()
    out = []
    for idx, sg, lut, n, g, e, on in ((ki, ks, par["lut_k"], sc[..., 0:1], sc[..., 1:2], ebar[:, 0], True),
                                      (vi, vs, par["lut_v"], sc[..., 2:3], sc[..., 3:4], ebar[:, 1], case["v_signs"])):
        x = torch.gather(lut[l].double()[:, None].expand(-1, idx.shape[1], -1), -1, idx)
        if on:
            x = x + (e[:, None, None] * sg if case["per_element"] else ALPHA * g * (sg @ S))
        out.append(x * (n / 8))
    return out


# ------------------------------------------------------------ raw inputs of a case
def _inputs(case, seed):
    """Everything a case's pass reads, as tensors, without the library's objects."""
    if case["op"].startswith("calibrate"):
        H, n = case["heads"], case["tokens"]
        g = _generator(seed, 4)
        scale = _outliers(case, seed)
        k, v = _kv(dict(case, layers=1, half_precision=False), g, scale, n)
        pos = torch.randint(0, 1024, (n,), generator=g, device=DEV)
        s = {"keys": _rope(k, pos, case["rope_half"])[0].transpose(0, 1).contiguous(), "values": v[0].transpose(0, 1).contiguous()}
        s["pi"] = _parameters(dict(case, layers=1), seed)["pi"][0].contiguous()
        return s
    L, B, H, T = case["layers"], case["batch"], case["heads"], case["tokens"]
    par = _parameters(case, seed)
    lens, first, slots = _lengths(case, seed)
    scale = _outliers(case, seed)
    io = torch.float16 if case["half_precision"] else torch.float32
    words = L * H * slots
    s = {"par": par, "lens": lens, "first": first, "slots": slots, "scale": scale,
         "cache": (torch.zeros(words * 32, dtype=torch.uint8, device=DEV),
                   torch.zeros(words * 32, dtype=torch.uint8, device=DEV),
                   torch.zeros(words * 4, dtype=torch.int16, device=DEV))}
    g = _generator(seed, 5)
    if case["op"].startswith("quantize"):
        s["k"] = torch.empty((L, B, T, H, D), dtype=io, device=DEV)
        s["v"] = torch.empty_like(s["k"])
        for b in range(B):
            s["k"][:, b], s["v"][:, b] = _kv(case, g, scale, T)
        cached = torch.full_like(lens, case["cached"])
        _fill(case, par, scale, seed, s["cache"], first, cached, slots)
    else:
        _fill(case, par, scale, seed, s["cache"], first, lens, slots)
        s["q"] = _randn(g, L, B, H, D).to(io)
        k, v = _kv(case, g, scale, B)
        s["k"], s["v"] = k.contiguous(), v.contiguous()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["op"].startswith("calibrate"):
        return s
    L, B, H = case["layers"], case["batch"], case["heads"]
    lens, cached = s["lens"], case["cached"]
    longest = int(lens.max()) + cached
    io = torch.float16 if case["half_precision"] else torch.float32
    s["params"] = tq.Params(L, H, tq.rope_table(longest + 64), io_dtype=io, flags=_flags(case))
    cache = tq.Cache(L, H, s["slots"])
    cache.k_codes, cache.v_codes, cache.scalars = s["cache"]
    s["cache"] = cache
    s["slot0"] = s["first"].to(DEV)
    s["len"] = lens.to(DEV, torch.int32)
    s["start"] = torch.full((B,), cached, dtype=torch.int32, device=DEV)
    s["start_slot"] = s["slot0"] + cached
    s["max_len"] = longest + (1 if case["op"] == "decode_step" else 0)
    if case["op"].startswith("decode"):
        need = tq.decode_workspace_bytes(s["params"], B, L, s["max_len"])
        s["workspace"] = torch.zeros(need, dtype=torch.uint8, device=DEV) if need else None
    if case["op"] == "dequantize":
        s["k_out"] = torch.zeros((L, B, H, longest, D), dtype=torch.float16, device=DEV)
        s["v_out"] = torch.zeros_like(s["k_out"])
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "calibrate_rotation":
        return tq.calibrate_rotation(s["keys"])
    if op == "calibrate_tables":
        pv = s["pi"] if case["v_rotate"] else None
        lut_k = tq.calibrate_lut(s["keys"], s["pi"])
        lut_v = tq.calibrate_lut(s["values"], pv)
        return (lut_k, lut_v, tq.calibrate_ebar(s["keys"], lut_k, s["pi"]), tq.calibrate_ebar(s["values"], lut_v, pv))
    par, cache = s["par"], s["cache"]
    tables = (par["pi"], par["lut_k"], par["lut_v"], par["S"])
    ebar = par["ebar"] if case["per_element"] else None
    if op == "decode_step":
        out = tq.decode_step(s["params"], cache, s["q"], s["k"], s["v"], s["len"], s["slot0"], s["len"], s["max_len"],
                             *tables, ebar=ebar, workspace=s["workspace"])
        return {"out": out, "k_codes": cache.k_codes, "v_codes": cache.v_codes,
                "scalars": cache.scalars.view(torch.float16)}
    if op == "decode_attend":
        return tq.decode_attend(s["params"], cache, s["q"], s["len"], s["slot0"], s["len"], s["max_len"], *tables,
                                ebar=ebar, workspace=s["workspace"])
    if op == "dequantize":
        return tq.dequantize(s["params"], cache, s["slot0"], s["len"], s["max_len"], par["lut_k"], par["lut_v"], par["S"],
                             ebar=ebar, k_out=s["k_out"], v_out=s["v_out"])
    tq.quantize_pack(s["params"], cache, s["k"], s["v"], s["start"], s["start_slot"], *tables, ebar=ebar,
                     seq_tokens=s["len"] if op == "quantize_ragged" else None)
    return {"k_codes": cache.k_codes, "v_codes": cache.v_codes, "scalars": cache.scalars.view(torch.float16)}


# ------------------------------------------------------------------ accounting
def _token_heads(case):
    """Expected token-heads of a pass (a ragged batch's lengths are uniform between shortest and tokens)."""
    mean = (case["shortest"] + case["tokens"]) / 2 if case["shortest"] else case["tokens"]
    return case["layers"] * case["heads"] * case["batch"] * mean


def work(case):
    H, n = case["heads"], case["tokens"]
    if case["op"] == "calibrate_rotation":
        return {"bytes": H * (n * D * 4 + D * D * 4 + D * 4), "flops": H * (n * D * (D + 1) + 10 * D ** 3)}
    if case["op"] == "calibrate_tables":
        turns = 2 if case["v_rotate"] else 1
        # the rotation once, and each sorted coordinate's share of the cell sums
        return {"bytes": H * (2 * n * D * 4 + D * D * 4 + 2 * 8 * 4 + 2 * 4),
                "flops": H * n * (turns * 2 * D * D + 2 * D * 8)}
    th = _token_heads(case)
    units = case["layers"] * H * case["batch"]
    io = 2 if case["half_precision"] else 4
    fixed = case["layers"] * H * (D * D * 4 + 64) + D * D * 4
    if case["op"] == "dequantize":
        return {"bytes": th * (72 + 4 * D) + fixed, "flops": th * (2 * D * D * (2 if case["v_signs"] else 1) + 6 * D)}
    if case["op"].startswith("quantize"):
        return {"bytes": th * (2 * D * io + 72) + fixed, "flops": th * (3 * 2 * D * D + 2 * 20 * D)}
    out = 2 if case["half_precision"] and not case["fp32_out"] else 4
    return {"bytes": th * 72 + fixed + units * (D * (io * (3 if case["op"] == "decode_step" else 1) + out) + 72),
            "flops": th * 6 * D + units * 2 * 3 * D * D}


def tolerance(case):
    """Set from the distance to exact() and from what sums in another order change."""
    op = case["op"]
    if op.startswith("calibrate"):                                 # fp64 inside: 2.5e-8 from 64 bits, the fp32 rounding
        return {"rel": 2e-7, "max": 1e-5}
    if op == "dequantize":
        return {"rel": 1e-4, "max": 4e-3}                          # fp16 rows: an ulp where rounding differs
    if op.startswith("quantize"):
        # A code or sign whose coordinate sits within rounding of its threshold (3e-6 of the coordinates
        # against 64 bits); fp16 norms by an ulp.
        return {"rel": 1e-4, "max": 4e-3, "differ": 1e-4}
    # fp32 outputs are 6e-7 from 64 bits; an appended code within rounding of its threshold moves its unit more.
    if case["half_precision"] and not case["fp32_out"]:
        return {"rel": 1e-4, "max": 8e-3, "differ": 1e-4}
    return {"rel": 1e-5, "max": 1e-3, "differ": 1e-4}


# ------------------------------------------------------------------ 64-bit results
def _exact_lloyd(x, pi, max_iter=100, tol=1e-7):
    u = _unit(x, pi)
    c = torch.tensor(GAUSS8, device=DEV).double().expand(u.shape[0], 8).contiguous()
    live = torch.ones(u.shape[0], dtype=torch.bool, device=DEV)
    for _ in range(max_iter):
        idx = torch.zeros(u.shape, dtype=torch.int64, device=DEV)
        for m in range(7):
            idx += u > 0.5 * (c[:, m:m + 1] + c[:, m + 1:m + 2])
        new = c.clone()
        for m in range(8):
            on = idx == m
            cnt = on.sum(1)
            new[:, m] = torch.where(cnt > 0, (u * on).sum(1) / cnt.clamp(min=1), c[:, m])
        delta = (new - c).abs().amax(1)
        c = torch.where(live[:, None], new.sort(1).values, c)
        live &= ~(delta < tol)
        if not bool(live.any()):
            break
    return c


def _unit(x, pi):
    y = x.double()
    if pi is not None:
        y = y @ pi.double().transpose(-1, -2).contiguous()
    n = y.norm(dim=-1, keepdim=True)
    return torch.where(n > 0, y * (8.0 / n), torch.zeros_like(y)).flatten(1)


def _exact_ebar(x, lut, pi):
    u, c = _unit(x, pi), lut.double()
    lv = c[:, :1].expand_as(u)
    for m in range(7):
        lv = torch.where(u > 0.5 * (c[:, m:m + 1] + c[:, m + 1:m + 2]), c[:, m + 1:m + 2], lv)
    return (u - lv).abs().mean(1)


def exact(case, seed):
    s = _inputs(case, seed)
    op = case["op"]
    if op == "calibrate_rotation":
        x = s["keys"].double()
        lam, vec = torch.linalg.eigh(x.transpose(1, 2).contiguous() @ x)
        pi = vec.flip(2).transpose(1, 2)
        big = torch.gather(pi, 2, pi.abs().argmax(2, keepdim=True))
        return pi * torch.where(big < 0, -1.0, 1.0), lam.flip(1).clamp(min=0).sqrt()
    if op == "calibrate_tables":
        pv = s["pi"] if case["v_rotate"] else None
        lk, lv = _exact_lloyd(s["keys"], s["pi"]), _exact_lloyd(s["values"], pv)
        return lk, lv, _exact_ebar(s["keys"], lk.float(), s["pi"]), _exact_ebar(s["values"], lv.float(), pv)
    par, L, H, B = s["par"], case["layers"], case["heads"], case["batch"]
    planes = _planes(case, s["cache"], s["slots"])
    sc = planes[2].double()
    lens, first = s["lens"].tolist(), s["first"].tolist()

    def layer(l):                                                  # one layer's parameters
        return {k: (v if k == "S" else v[l:l + 1]) for k, v in par.items()}

    if op.startswith("quantize"):
        for l in range(L):
            for b in range(B):
                n, at = lens[b], first[b] + case["cached"]
                pos = torch.arange(case["cached"], case["cached"] + n)
                kq, vq = _quantize_kv(case, layer(l), s["k"][l:l + 1, b, :n].double(), s["v"][l:l + 1, b, :n].double(), pos)
                sc[l:l + 1, :, at:at + n] = torch.stack([kq[2], kq[3], vq[2], vq[3]], -1).transpose(1, 2)
        return {"k_codes": None, "v_codes": None, "scalars": sc.flatten()}
    if op == "dequantize":
        rows = torch.zeros((2, L, B, H, max(lens), D), dtype=torch.float64, device=DEV)
        for l in range(L):
            for b in range(B):
                k, v = _rows(case, par, l, _unpack(planes, l, first[b], lens[b]))
                rows[0, l, b, :, :lens[b]], rows[1, l, b, :, :lens[b]] = k, v
        return rows[0], rows[1]
    out = torch.zeros((L, B, H, D), dtype=torch.float64, device=DEV)
    for l in range(L):
        for b in range(B):
            n = lens[b]
            if op == "decode_step":                                # append, then attend over n + 1 tokens
                new = _quantize_kv(case, layer(l), s["k"][l:l + 1, b:b + 1].double(), s["v"][l:l + 1, b:b + 1].double(),
                                   torch.tensor([n]))
                sc[l, :, first[b] + n] = torch.stack([new[0][2], new[0][3], new[1][2], new[1][3]], -1)[0, 0]
                (ki, kb, kn, kg), (vi, vb, vn, vg) = ([t[0].movedim(0, 1) for t in q] for q in new)
                tail = (ki, kb.double() * 2 - 1, vi, vb.double() * 2 - 1,
                        torch.stack([kn, kg, vn, vg], -1).half().double())
                codes = [torch.cat([a, t], 1) for a, t in zip(_unpack(planes, l, first[b], n), tail)]
            else:
                codes = _unpack(planes, l, first[b], n)
            k, v = _rows(case, par, l, codes)
            pi = par["pi"][l].double()
            q = _rope(s["q"][l, b].double()[None], torch.tensor([n]), case["rope_half"])[0]
            qr = (pi * q[:, None, :]).sum(-1)
            w = torch.softmax((k * qr[:, None, :]).sum(-1) * 0.125, -1)
            o = (w[..., None] * v).sum(1)
            out[l, b] = (pi * o[:, :, None]).sum(1) if case["v_rotate"] else o
    return {"out": out, "k_codes": None, "v_codes": None, "scalars": sc.flatten()} if op == "decode_step" else out
