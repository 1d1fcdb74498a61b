"""The workloads whose speed is watched: the framework's main path (quantize, forward, matched or stale correction, backward) called as a
training program calls it, over the range of sizes, head shapes, types and options the entry points take.

A case is a dict of plain values:
  op      "quantize"   one operand's MX copies and channel maxima
          "producer"   QK normalization, rotary embedding, prescale, key centring, then the quantizer
          "forward"    the attention forward on quantized operands
          "backward"   the whole backward call (correction, main pass, dQ) on quantized operands
          "attention"  forward then backward on quantized operands
          "step"       a training step: quantize Q, K, V, dO, forward, backward
  B, N, Nk, Hq, Hkv, dqk, dv, causal   the problem
  dtype   storage type of Q, K, V, dO ("bf16" / "f32"; O and the gradients have the same)
  dist    input recipe: "normal"; "outlier" (one channel of Q and K x3: its products
          dominate the scores, and rows do not become one-hot, whose gradients cancel to nothing); "qknorm" (RMS-normalized rows with gains U(0.5, 2));
          "rope" (rotary part on the last 64 channels, shared by the heads of K); "temperature" (query rows x U(0.5, 3))
  mode    row correction: "matching", "stale", "consistent"
  lens    sequences of a padded batch take the lengths N, 3N/4, N/2, N/4, N, .. (causal), rounded down to 32
"""
import math

import torch

import paper_2609_37852_amd as pk

MODES = {"matching": pk.DELTA_MATCHING, "stale": pk.DELTA_STALE_ROWSUM, "consistent": pk.DELTA_CONSISTENT_DO}
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(op, B, N, Hq, Hkv, dqk, dv, dist="normal", causal=True, Nk=0, dtype="bf16", mode="matching", lens=False, **kw):
    return dict(op=op, B=B, N=N, Nk=Nk or N, Hq=Hq, Hkv=Hkv, dqk=dqk, dv=dv, causal=causal, dtype=dtype, dist=dist, mode=mode, lens=lens,
                **kw)


def listed():
    return [
        # the smallest training step (2 heads of 64, 128 tokens, FP32): latency, launches and host work
        _case("step", 1, 128, 2, 2, 64, 64, dtype="f32", name="step tiny f32"),
        # one short sequence, a ragged 65 blocks of 32 tokens, 16 / 4 heads: a chip that one problem does not fill
        _case("step", 1, 2080, 16, 4, 128, 128, "outlier", name="step 2080 d128"),
        # the benchmark's step: 4 x 8192 tokens, 16 / 4 heads of 128, an outlier channel
        _case("step", 4, 8192, 16, 4, 128, 128, "outlier", name="step 8k d128"),
        # the query operand of that step
        _case("quantize", 4, 8192, 16, 4, 128, 128, "outlier", name="quantize 8k d128"),
        # its key operand through the producer: norm, rotation of 64 channels, centring
        _case("producer", 4, 8192, 4, 4, 128, 128, rope=64, center=True, name="producer key 8k d128"),
        # inference or the forward half of training on it
        _case("forward", 4, 8192, 16, 4, 128, 128, "outlier", name="forward 8k d128"),
        # cross attention: no mask, a key length of its own, small heads, FP32 outputs, ragged lengths
        _case("attention", 3, 1056, 8, 2, 64, 64, causal=False, Nk=2784, dtype="f32", name="cross 1056x2784 d64 f32"),
        # wide heads with QK normalization
        _case("attention", 2, 8192, 8, 2, 256, 256, "qknorm", name="attention 8k d256"),
        # MLA-shaped heads, 32 of them without grouping
        _case("attention", 2, 4096, 32, 32, 192, 128, "rope", name="attention mla 4k d192"),
        # the saved-output correction, the baseline of the matched one
        _case("backward", 4, 4096, 16, 4, 128, 128, mode="stale", name="backward stale 4k d128"),
        # a padded batch of sequences of 8192, 6144, 4096 and 2048 tokens
        _case("attention", 4, 8192, 16, 4, 128, 128, "outlier", lens=True, name="attention varlen d128"),
        # one long document
        _case("backward", 1, 65536, 16, 4, 128, 128, "temperature", name="backward 64k d128"),
    ]


def draw(rng):
    def size(lo, hi):      # a multiple of 32, spread over the logarithm
        return max(1, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 32)) * 32

    op = rng.choice(["step", "step", "quantize", "producer", "forward", "backward", "attention", "attention"])
    dqk, dv = rng.choice([(64, 64), (128, 128), (128, 128), (192, 128), (256, 256)])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    B, Hkv = rng.randint(1, 4), rng.choice([1, 2, 3, 4, 8])
    Hq = Hkv * rng.choice([1, 2, 4, 5])
    N = size(32, 8192)
    if op == "quantize":
        return _case(op, B, N, Hq, Hkv, dqk, dv, rng.choice(["normal", "outlier"]), dtype=dtype)
    if op == "producer":
        return _case(op, B, N, Hkv, Hkv, dqk, dv, dtype=dtype, rope=rng.choice([0, 32, 64]), center=rng.random() < 0.7)
    while B * Hq * N * N > 4 * 16 * 8192 * 8192 // 2:   # at most half of the benchmark's pairs
        N = N // 64 * 32
    causal = rng.random() < 0.75
    Nk = N if causal else size(32, 4096)
    dist = "rope" if dqk == 192 else rng.choice(["normal", "outlier", "temperature", "qknorm"])
    # a saved-output correction of sharply peaked rows cancels almost wholly: it meets the milder recipes
    mode = "matching" if dist in ("outlier", "temperature") else rng.choice(["matching", "matching", "stale", "consistent"])
    return _case(op, B, N, Hq, Hkv, dqk, dv, dist, causal, Nk, dtype, mode, lens=causal and B > 1 and N >= 256 and rng.random() < 0.25)


# --- inputs -----------------------------------------------------------------

def _inputs(c, seed):
    """Raw Q, K, V, dO of a case, [B, L, H, D] of its type on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    B, N, Nk = c["B"], c["N"], c["Nk"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

    def uniform(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(shape, generator=g, device="cuda", dtype=torch.float32)

    q, k = normal(B, N, c["Hq"], c["dqk"]), normal(B, Nk, c["Hkv"], c["dqk"])
    v, do = normal(B, Nk, c["Hkv"], c["dv"]), normal(B, N, c["Hq"], c["dv"])
    if c["dist"] == "outlier":
        ch = int(torch.randint(c["dqk"], (1,), generator=g, device="cuda"))
        q[..., ch] *= 3.0
        k[..., ch] *= 3.0
    elif c["dist"] == "qknorm":
        gains = uniform(0.5, 2.0, 2, c["dqk"])
        q, k = (x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-6) * y for x, y in zip((q, k), gains))
    elif c["dist"] == "rope":
        k[..., -64:] = normal(B, Nk, 1, 64)
        for x in (q, k):
            cs = _rope_table(x.shape[1], 64)
            a, b = x[..., -64:-32].clone(), x[..., -32:].clone()
            cos, sin = cs[None, :, None, :, 0], cs[None, :, None, :, 1]
            x[..., -64:-32], x[..., -32:] = a * cos - b * sin, b * cos + a * sin
    elif c["dist"] == "temperature":
        q *= uniform(0.5, 3.0, B, N, c["Hq"], 1)
    return tuple(x.to(DTYPES[c["dtype"]]) for x in (q, k, v, do))


def _rope_table(n, r):
    """[n, r / 2, 2] float32 cosines and sines, base 10000."""
    ang = torch.arange(n, device="cuda", dtype=torch.float64)[:, None] * 10000.0 ** (
        -torch.arange(r // 2, device="cuda", dtype=torch.float64)[None, :] * 2.0 / r)
    return torch.stack([ang.cos(), ang.sin()], -1).float().contiguous()


def _gain(c, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 7)
    return 0.5 + 1.5 * torch.rand((c["dqk"],), generator=g, device="cuda", dtype=torch.float32)


def _lens(c):
    return [max(32, c["N"] * (4 - b % 4) // 4 // 32 * 32) for b in range(c["B"])] if c["lens"] else [c["N"]] * c["B"]


def _tau(c):
    return float(torch.tensor(1.0 / math.sqrt(c["dqk"]), dtype=torch.float32))


# --- the calls --------------------------------------------------------------

def _quantize_all(q, k, v, do=None):
    """The operands' MX copies; channel maxima for Q and K only (nothing reads those of V and dO)."""
    m = [pk.attn_fp8_quantize(q), pk.attn_fp8_quantize(k), pk.attn_fp8_quantize(v, amax=False)]
    return m if do is None else m + [pk.attn_fp8_quantize(do, amax=False)]


def prepare(case, seed):
    c, op = case, case["op"]
    q, k, v, do = _inputs(c, seed)
    if op == "quantize":
        return dict(c=c, x=q)
    if op == "producer":
        return dict(c=c, x=k, gain=_gain(c, seed), rope=_rope_table(c["N"], c["rope"]) if c["rope"] else None)
    lens = torch.tensor(_lens(c), dtype=torch.int32, device="cuda") if c["lens"] else None
    p = pk.Problem(c["B"], c["N"], c["Hq"], c["Hkv"], c["dqk"], c["dv"], _tau(c), causal=int(c["causal"]),
                   seqlen_kv=0 if c["causal"] else c["Nk"], seqlens_q=lens)
    dt = DTYPES[c["dtype"]]
    # the buffers of a program that keeps them between steps (the padding of a padded batch stays zero)
    s = dict(c=c, p=p, raw=(q, k, v, do), o=torch.zeros_like(do), lse=torch.zeros((c["B"], c["Hq"], c["N"]), device="cuda"),
             grads=(torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)), dt=dt)
    if op != "forward":
        s["ws"] = torch.empty(max(pk.attn_fp8_bwd_workspace_size(p), 256), dtype=torch.uint8, device="cuda")
    if op != "step":
        s["mx"] = _quantize_all(q, k, v) if op == "forward" else _quantize_all(q, k, v, do)
    if op == "backward":
        pk.attn_fp8_fwd(p, *s["mx"][:3], o=s["o"], lse=s["lse"])
    return s


def run(state):
    s, c, op = state, state["c"], state["c"]["op"]
    if op == "quantize":
        return _mx_out(pk.attn_fp8_quantize(s["x"]))
    if op == "producer":
        m, mean = pk.attn_fp8_quantize_producer(s["x"], center=c["center"], rope=s["rope"], rms_gain=s["gain"])
        return _mx_out(m) + ([mean] if c["center"] else [])
    mx = _quantize_all(*s["raw"]) if op == "step" else s["mx"]
    out = []
    if op != "backward":
        out += pk.attn_fp8_fwd(s["p"], *mx[:3], o=s["o"], lse=s["lse"])
    if op != "forward":
        raw = dict(dout_raw=s["raw"][3], o=s["o"]) if c["mode"] != "matching" else {}
        out += pk.attn_fp8_bwd(s["p"], MODES[c["mode"]], *mx, s["lse"], workspace=s["ws"], out=s["grads"], **raw)[:3]
    return out


def _mx_out(m):
    return [m.code_row, m.scale_row, m.code_col, m.scale_col, m.channel_amax]


# --- what a pass needs, and what it should give -----------------------------

def work(case):
    c, es = case, 2 if case["dtype"] == "bf16" else 4
    q, k = c["B"] * c["N"] * c["Hq"] * c["dqk"], c["B"] * c["Nk"] * c["Hkv"] * c["dqk"]
    o, v = c["B"] * c["N"] * c["Hq"] * c["dv"], c["B"] * c["Nk"] * c["Hkv"] * c["dv"]
    mx = 2 * (1 + 1 / 32)                    # bytes an element of both MX copies
    if c["op"] == "quantize":
        return {"bytes": q * (es + mx), "flops": 4 * q}
    if c["op"] == "producer":
        return {"bytes": k * (es + mx) + 4 * c["N"] * c["rope"], "flops": 12 * k}
    pairs = c["Hq"] * sum(n * (n + 1) // 2 if c["causal"] else n * c["Nk"] for n in _lens(c))
    lse = 4 * c["B"] * c["Hq"] * c["N"]
    fwd, bwd = 2 * pairs * (c["dqk"] + c["dv"]), 2 * pairs * (3 * c["dqk"] + 2 * c["dv"])
    one = mx / 2                             # a product reads one of an operand's two copies
    by = {"forward": (q + k + v) * one + o * es + lse,
          "backward": (q + k + o) * mx + v * one + lse + (q + k + v) * es + (2 * o * es if c["mode"] == "stale" else 0)}
    by["attention"] = (q + k + o + v) * mx + o * es + lse + (q + k + v) * es
    by["step"] = (q + k + v + o) * es + o * es + lse + (q + k + v) * es
    flops = {"forward": fwd, "backward": bwd, "attention": fwd + bwd, "step": fwd + bwd}[c["op"]]
    share = sum(_lens(c)) / (c["B"] * c["N"])   # rows inside their sequences
    return {"bytes": by[c["op"]] * share, "flops": flops}


def tolerance(case):
    # the quantizer and the producer give bytes, and sums in a stated order.  The attention's P and dS are cast to E4M3, so sums in another
    # order move codes by one step (6 %) here and there: against the same casts in 64 bits the outputs are 1e-4 to 5e-3 off, single values up
    # to 0.6 of the root mean square where one element carries its gradient.
    if case["op"] in ("quantize", "producer"):
        return "exact"
    return {"rel": 2e-2, "max": 0.99}


# --- the same in 64 bits ----------------------------------------------------

def _pow2_exponent(amax):
    """Smallest e with amax <= 448 * 2^e, in [-127, 127]; zero and subnormal amax give -127."""
    m, e = torch.frexp(amax.double() / 448.0)          # m in [0.5, 1): 2^e > x, and x = 2^(e - 1) where m = 0.5
    e = torch.where(m == 0.5, e - 1, e)
    return torch.where(amax.double() < 2.0 ** -126, torch.full_like(e, -127), e).clamp(-127, 127)


def _e4m3(x):
    return x.float().to(torch.float8_e4m3fn).double()


def _cast(x, dim):
    """x quantized to E4M3 with one power-of-two scale for each 32 values along dim (0 or 1 of a matrix), decoded."""
    y = x.double() if dim == 1 else x.double().t()
    b = y.reshape(y.shape[0], y.shape[1] // 32, 32)
    s = torch.ldexp(torch.ones((), dtype=torch.float64, device=x.device), _pow2_exponent(b.abs().amax(-1, keepdim=True)))
    y = (_e4m3(b / s) * s).reshape(y.shape)
    return y if dim == 1 else y.t().contiguous()


def _head(c, q, do, o, K, V, tau, n):
    """One query head over its n (causal) queries: O, LSE, dQ, and its part of dK, dV (for 1 query head), FP8 casts included."""
    qr, qc = _cast(q, 1), _cast(q, 0)
    dr, dc = _cast(do, 1), _cast(do, 0)
    Kr, Kc, Vr, Vc = K["row"], K["col"], V["row"], V["col"]
    nk = Kr.shape[0]
    O, dQ = torch.empty((n, Vr.shape[1]), dtype=torch.float64, device=q.device), torch.empty_like(qr)
    lse = torch.empty((n,), dtype=torch.float64, device=q.device)
    dK, dV = torch.zeros_like(Kr), torch.zeros_like(Vr)
    rows = max(32, (1 << 26) // nk // 32 * 32)
    for r0 in range(0, n, rows):
        r1 = min(n, r0 + rows)
        e = r1 if c["causal"] else nk
        x = tau * qr[r0:r1] @ Kr[:e].t()
        mask = None
        if c["causal"]:
            mask = torch.arange(e, device=q.device)[None, :] > torch.arange(r0, r1, device=q.device)[:, None]
            x = x.masked_fill(mask, -math.inf)
        L = torch.logsumexp(x, -1)
        p = torch.exp(x - L[:, None])
        lse[r0:r1] = L
        if c["op"] != "backward":
            # codes of 2^(x log2 e) for each row's 32 keys, with the smallest E that keeps them at most 448
            g = (x * math.log2(math.e)).reshape(r1 - r0, e // 32, 32)
            E = torch.ceil(g.amax(-1, keepdim=True) - math.log2(448.0))
            E = torch.where(torch.isfinite(E), E, torch.zeros_like(E))
            ph = _e4m3(torch.exp2(g - E)) * torch.exp2(E - (L * math.log2(math.e))[:, None, None])
            O[r0:r1] = ph.reshape(r1 - r0, e) @ Vc[:e]
            del g, ph
        if c["op"] == "forward":
            continue
        dp = dr[r0:r1] @ Vr[:e].t()
        if c["mode"] == "matching":
            delta = (p * dp).sum(-1) / p.sum(-1)
        else:
            delta = ((do if c["mode"] == "stale" else dr)[r0:r1].double() * o[r0:r1].double()).sum(-1)
        ds = p * (dp - delta[:, None])
        del dp, x
        b = ds.reshape((r1 - r0) // 32, 32, e // 32, 32)
        sc = torch.ldexp(torch.ones((), dtype=torch.float64, device=q.device), _pow2_exponent(b.abs().amax((1, 3), keepdim=True)))
        ds = (_e4m3(b / sc) * sc).reshape(r1 - r0, e)
        ph = _e4m3(p * 256.0) / 256.0
        dV[:e] += ph.t() @ dc[r0:r1]
        dK[:e] += tau * (ds.t() @ qc[r0:r1])
        dQ[r0:r1] = tau * (ds @ Kc[:e])
    return O, lse, dQ, dK, dV


def exact(case, seed):
    c = case
    if c["op"] == "quantize":
        x = _inputs(c, seed)[0]
        return [None, None, None, None, x.double().abs().amax(1)]
    if c["op"] == "producer":
        # the normalization and the rotation are defined with FP32 and bfloat16 roundings between their steps; the sums are taken in 64 bits
        x = _inputs(c, seed)[1]
        r = (1.0 / torch.sqrt(x.double().square().mean(-1, keepdim=True) + float(torch.tensor(1e-6)))).float()
        y = (x.float() * r * _gain(c, seed)).bfloat16().float()
        if c["rope"]:
            h = c["rope"] // 2
            cos, sin = _rope_table(c["N"], c["rope"])[None, :, None].unbind(-1)
            a, b = y[..., :h].clone(), y[..., h:2 * h].clone()
            y[..., :h], y[..., h:2 * h] = (a * cos - b * sin).bfloat16().float(), (b * cos + a * sin).bfloat16().float()
        mean = y.double().mean(1)
        if not c["center"]:
            return [None, None, None, None, y.double().abs().amax(1)]
        return [None, None, None, None, (y.double() - mean[:, None]).abs().amax(1), mean]
    tau = _tau(c)
    q, k, v, do = _inputs(c, seed)
    f64 = dict(dtype=torch.float64, device="cuda")
    O, lse = torch.zeros(do.shape, **f64), torch.zeros((c["B"], c["Hq"], c["N"]), **f64)
    dQ, dK, dV = (torch.zeros(x.shape, **f64) for x in (q, k, v))
    sub = dict(c, op="attention") if c["mode"] != "matching" else c
    for b, n in enumerate(_lens(c)):
        nk = n if c["causal"] else c["Nk"]
        for h in range(c["Hq"]):
            kh = h // (c["Hq"] // c["Hkv"])
            K, V = k[b, :nk, kh], v[b, :nk, kh]
            K, V = ({"row": _cast(x, 1), "col": _cast(x, 0)} for x in (K, V))
            qh, dh, o = q[b, :n, h], do[b, :n, h], None
            if c["mode"] != "matching":     # the stored output, in its type
                o = _head(dict(c, op="forward"), qh, dh, None, K, V, tau, n)[0].to(DTYPES[c["dtype"]])
            r = _head(sub, qh, dh, o, K, V, tau, n)
            O[b, :n, h], lse[b, h, :n], dQ[b, :n, h] = r[0], r[1], r[2]
            dK[b, :nk, kh] += r[3]
            dV[b, :nk, kh] += r[4]
    fwd, bwd = [O, lse], [dQ, dK, dV]
    return {"forward": fwd, "backward": bwd}.get(c["op"], fwd + bwd)
