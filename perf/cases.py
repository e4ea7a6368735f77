"""The work that a user of this framework has it do, as cases that can be timed and checked.

A case is a dict of plain values.  `prepare` makes what a drafting program has in hand before the call
(caches, weights, lengths, output buffers), `run` is one pass through the public entry points, `exact`
the same results in 64 bits by plain torch.  Inputs are synthetic: N(0, 1) activations, queries, keys and
values, N(0, 0.02^2) weights, N(0, 1) logits with planted acceptance, softmax(N(0, 1) / 0.5) distributions.

Kinds of case (`kind`):
  decode    one token of B sequences through the draft's attention: sinks + slots, the local window, the
            new token, which is appended (`full`: the uncompressed comparison, the whole prefix as window)
  boundary  the same for a pass in which sequences materialise slots: memory update, then the attention
  step      one sequence's fused boundary pass: memory update, then the raw query and the new slots'
            write scopes in one launch
  verify    the target's T-query attention over its full KV (`vt`: V stored key-contiguous)
  greedy    greedy accept/reject over the target's logits
  stoch     stochastic accept/reject over target and draft distributions
  prefill   the draft's masked attention over a whole prefix, slot queries included
  layer     one decoder layer of the draft for a token (rows > 1: with the slots made in its pass)
  maps      the four linear maps of a draft layer alone
"""
import math
import random

import torch

import paper_2608_30252_amd as mad
from paper_2608_30252_amd.layer import DraftLayer, LayerWeights
from paper_2608_30252_amd.state import MemoryLayout

DEV = "cuda"
ROPE_BASE = 500000.0
EPS = 1e-5
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest call of a draft loop: one sequence, an 8K prefix as 512 slots + a 512-token window
        dict(name="decode_8k", kind="decode", B=1, Hq=32, Hkv=8, d=64, dtype="bf16", S=0, W=512, r=16, u=4, lo=8192,
             hi=8192, lens=1, full=False),
        # a serving batch: 64 sequences of ragged prefixes, 128 sinks, each at its own memory length
        dict(name="decode_batch64", kind="decode", B=64, Hq=32, Hkv=8, d=64, dtype="bf16", S=128, W=1024, r=16, u=4,
             lo=2048, hi=32768, lens=2, full=False),
        # the uncompressed comparison with the heads of an 8B-shaped model: the whole prefix per token
        dict(name="decode_full_d128", kind="decode", B=4, Hq=32, Hkv=8, d=128, dtype="bf16", S=0, W=32768, r=16, u=1,
             lo=16000, hi=32000, lens=3, full=True),
        # batched drafting at a block end: 16 ragged sequences, 4 slots each, half of them firing
        dict(name="boundary_batch16", kind="boundary", B=16, Hq=32, Hkv=8, d=64, dtype="bf16", S=0, W=512, r=16, u=4,
             lo=8192, hi=32768, lens=4, D=2048),
        # the fp32 form of the same pass (parity and numerics work), the paper's S = W = 128 and r = 4
        dict(name="boundary_f32", kind="boundary", B=4, Hq=32, Hkv=8, d=64, dtype="f32", S=128, W=128, r=4, u=4,
             lo=2048, hi=8192, lens=5, D=2048),
        # the target's verification at a long prefix: an 8B-shaped layer, 4 sequences, gamma = 4
        dict(name="verify_8b_32k", kind="verify", B=4, T=5, Hq=32, Hkv=8, d=128, dtype="bf16", lo=32768, hi=32768,
             lens=6, vt=False),
        # a serving batch in verification: ragged prefixes, 8 query heads per KV head, gamma = 5
        dict(name="verify_ragged16", kind="verify", B=16, T=6, Hq=64, Hkv=8, d=128, dtype="bf16", lo=600, hi=12000,
             lens=7, vt=False),
        # accepting a drafted block of 16 sequences over a 128256-token vocabulary
        dict(name="greedy_batch16", kind="greedy", B=16, T=5, V=128256, dtype="f32"),
        # rejection sampling for a batch over a vocabulary with no alignment
        dict(name="stoch_batch16", kind="stoch", B=16, T=6, V=50257),
        # the draft's prefill of a 32K prefix with its 2048 slots
        dict(name="prefill_32k", kind="prefill", B=1, Hq=32, Hkv=8, d=64, S=0, W=1024, r=16, u=4, lo=32768, hi=32768,
             lens=10),
        # a batch of shorter, ragged prefixes at head_dim 128, the paper's S = W = 128 with r = 8
        dict(name="prefill_ragged_d128", kind="prefill", B=4, Hq=32, Hkv=8, d=128, S=128, W=128, r=8, u=1, lo=2000,
             hi=8000, lens=11),
        # a draft layer for one token at a 32K prefix: five dependent launches around a weight stream
        dict(name="layer_32k", kind="layer", D=2048, Hq=32, Hkv=8, d=64, F=8192, S=0, W=1024, r=16, u=4, p=32700,
             rows=1),
    ]


# ------------------------------------------------------------------ draws ----

def _logu(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode"] * 4 + ["boundary", "boundary", "step", "verify", "verify", "verify", "greedy", "stoch",
                                        "prefill", "prefill", "layer", "layer", "maps"])
    lens = rng.randrange(1, 1 << 20)
    if kind in ("decode", "boundary", "step"):
        Hkv, G = rng.choice([(8, 4), (8, 4), (8, 4), (8, 8), (8, 1), (8, 2), (2, 16), (4, 4)])
        d = rng.choice([64, 64, 128])
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        S, W, r, u = rng.choice([(0, 512, 16, 4), (0, 1024, 16, 4), (128, 128, 4, 4), (128, 128, 8, 1), (4, 300, 8, 1)])
        B = 1 if kind == "step" else _logu(rng, 1, 64 // u if kind == "boundary" else 64)
        full = kind == "decode" and rng.random() < 0.25
        row = Hkv * d * 2 * (2 if dtype == "bf16" else 4)
        most = 32768 if not full else min(32768, max(256, 500_000_000 // (B * row)))
        hi = _logu(rng, 256, most)
        c = dict(kind=kind, B=B, Hq=Hkv * G, Hkv=Hkv, d=d, dtype=dtype, S=S, W=W, r=r, u=u,
                 lo=max(192, hi // rng.choice([1, 2, 8])), hi=hi, lens=lens)
        if kind == "decode":
            c["full"] = full
        else:
            c["D"] = rng.choice([1536, 2048, 4096])
        return c
    if kind == "verify":
        Hkv, G = rng.choice([(8, 4), (8, 4), (8, 8), (8, 1), (2, 16)])
        d, dtype = rng.choice([64, 128, 128]), rng.choice(["bf16", "bf16", "bf16", "bf16", "f32"])
        T = rng.randrange(1, min(8, 64 // G) + 1)
        B = _logu(rng, 1, 32 if dtype == "bf16" else 4)
        row = Hkv * d * 2 * (2 if dtype == "bf16" else 4)
        hi = _logu(rng, 300, min(32768, 500_000_000 // (B * row)))
        return dict(kind=kind, B=B, T=T, Hq=Hkv * G, Hkv=Hkv, d=d, dtype=dtype, lo=max(64, hi // rng.choice([1, 2, 8])),
                    hi=hi, lens=lens, vt=dtype == "bf16" and rng.random() < 0.3)
    if kind == "greedy":
        T = rng.randrange(2, 8)
        return dict(kind=kind, B=_logu(rng, 1, 32), T=T, V=_vocab(rng), dtype=rng.choice(["bf16", "f32"]))
    if kind == "stoch":
        return dict(kind=kind, B=_logu(rng, 1, 32), T=rng.randrange(2, 8), V=_vocab(rng))
    if kind == "prefill":
        Hkv, G = rng.choice([(8, 4), (8, 4), (8, 8), (8, 1), (4, 2)])
        d = rng.choice([64, 128])
        S, W, r, u = rng.choice([(0, 512, 16, 4), (0, 1024, 16, 4), (128, 128, 4, 4), (128, 128, 8, 1), (4, 300, 8, 1)])
        B = _logu(rng, 1, 8)
        hi = _logu(rng, 200, 12000 // B if G * d <= 256 else 6000 // B)
        return dict(kind=kind, B=B, Hq=Hkv * G, Hkv=Hkv, d=d, S=S, W=W, r=r, u=u, lo=max(100, hi // rng.choice([1, 2, 8])),
                    hi=hi, lens=lens)
    if kind == "layer":
        D, d = rng.choice([(2048, 64), (2048, 64), (4096, 128)])
        S, W, r, u = rng.choice([(0, 512, 16, 4), (0, 1024, 16, 4), (128, 128, 4, 4), (128, 128, 8, 1)])
        p = _logu(rng, 300, 32000)
        rows = rng.choice([1, 1 + u])
        blk = r * u
        if rows > 1:      # the last token of a block, whose pass makes u slots
            p = S + (p - S) // blk * blk + blk - 1
        elif (p - S + 1) % blk == 0:
            p += 1
        return dict(kind=kind, D=D, Hq=32, Hkv=8, d=d, F=rng.choice([4096, 8192]), S=S, W=W, r=r, u=u, p=p, rows=rows)
    D, d = rng.choice([(2048, 64), (4096, 128)])
    return dict(kind="maps", D=D, Hq=32, Hkv=8, d=d, F=rng.choice([4096, 8192]), rows=rng.randrange(1, 9),
                pos=rng.randrange(100, 32768))


def _vocab(rng):
    return rng.choice([_logu(rng, 4000, 160000), _logu(rng, 4000, 160000) // 64 * 64, 128256])


# ---------------------------------------------------------------- lengths ----

def _prefixes(c):
    rng = random.Random(c["lens"])
    return [c["hi"] if c["B"] == 1 else rng.randint(c["lo"], c["hi"]) for _ in range(c["B"])]


def _slots(t, c):
    """Slots materialised once raw tokens 0 .. t-1 are processed."""
    return 0 if t <= c["S"] else (t - c["S"]) // (c["r"] * c["u"]) * c["u"]


def _ring_cap(c):
    return c["W"] + 5 + 16 + c["r"] * c["u"]


def _win(c, lo, hi, cap):
    """(length, ring start) of raw positions [lo, hi)."""
    lo = max(c["S"], lo)
    return max(0, hi - lo), (lo - c["S"]) % cap


def _views(c):
    """Per sequence (memory rows, window rows, ring start) of the token at its prefix's end, which is appended."""
    cap, out = _ring_cap(c), []
    for p in _prefixes(c):
        if c.get("full"):
            out.append((0, p - 1, 0))
        else:
            p = max(p, c["S"] + 1)
            n, st = _win(c, p - c["W"] + 1, p, cap)
            out.append((c["S"] + _slots(p, c), n, st))
    return out


def _block_end(c, p):
    blk = c["r"] * c["u"]
    return c["S"] + max(1, (p - c["S"]) // blk) * blk - 1


def _boundary_views(c):
    """As _views for tokens at a block's end, and the position ids of the slots made in their pass."""
    cap, out, pos = _ring_cap(c), [], []
    for p in _prefixes(c):
        p = _block_end(c, p)
        n, st = _win(c, p - c["W"] + 1, p, cap)
        before = _slots(p, c)
        out.append((c["S"] + before, n, st))
        pos.append([c["S"] + (before + 1 + i) * c["r"] for i in range(c["u"])])
    return out, pos


def _step_views(c):
    """Rows of one sequence's fused boundary pass at position p: (memory rows, window rows, ring start, mode)."""
    cap = _ring_cap(c)
    p = _block_end(c, c["hi"])
    n, st = _win(c, p - c["W"] + 1, p, cap)
    before = _slots(p, c)
    rows, pos = [(c["S"] + before, n, st, 2)], []
    for i in range(c["u"]):
        b = c["S"] + (before + 1 + i) * c["r"]
        n, st = _win(c, b - c["W"], b, cap)
        last = b - 1 == p
        rows.append((c["S"] + before + 1 + i, n - 1 if last else n, st, 1 if last else 0))
        pos.append(b)
    return rows, pos


def _fire(c):
    return [1 if (b + c["lens"]) % 2 == 0 or c["B"] < 4 else 0 for b in range(c["B"])]


# ---------------------------------------------------------------- prepare ----

class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)

    def normal(self, shape, dtype, std=1.0, mean=0.0):
        return (torch.randn(shape, generator=self.g, device=DEV, dtype=torch.float32) * std + mean).to(dtype)


def prepare(c, seed):
    g, k = _Gen(seed), c["kind"]
    dt = DTYPES[c.get("dtype", "bf16")]
    B, Hq, Hkv, d = c.get("B", 1), c.get("Hq"), c.get("Hkv"), c.get("d")
    s = {"kind": k}
    if k in ("decode", "boundary", "step"):
        rows = c["u"] + 1 if k == "step" else B
        if k == "decode":
            views = _views(c)
        elif k == "boundary":
            views, s["pos"] = _boundary_views(c)
            s["fire"] = _fire(c)
        else:
            views, pos = _step_views(c)
            s["pos"], s["modes"] = [pos], [v[3] for v in views]
        cap = max(v[1] for v in views) + 21 if c.get("full") else _ring_cap(c)
        mcap = max(v[0] for v in views) + c["u"]
        s["views"] = views
        s["q"] = g.normal((rows, Hq, d), dt)
        kn, vn = g.normal((B, Hkv, d), dt), g.normal((B, Hkv, d), dt)
        s["kn"], s["vn"] = (t.expand(rows, Hkv, d).contiguous() if k == "step" else t for t in (kn, vn))
        ring = [g.normal((B, Hkv, cap, d), dt) for _ in range(2)]
        s["ring"] = ring
        starts = [v[2] for v in views]
        if c.get("full"):
            s["mem"], s["mem_kv"] = None, None
        else:
            s["mem"] = [g.normal((B, Hkv, mcap, d), dt) for _ in range(2)]
            seen = [v[0] for v in views]
            if k == "boundary":     # the token's own pass attends the slots that existed before it
                s["upd_kv"] = mad.KV(*s["mem"], [v[0] for v in views])
            elif k == "step":
                s["upd_kv"] = mad.KV(*s["mem"], [views[0][0]])
            s["mem_kv"] = mad.KV(*s["mem"], seen)
        s["ring_kv"] = mad.KV(*ring, [v[1] for v in views], starts)
        if k != "decode":
            s["x"] = g.normal((B, c["u"], c["D"]), dt)
            s["w"] = g.normal((2 * Hkv * d, c["D"]), dt, std=0.02)
        s["out"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((rows, Hq), dtype=torch.float32, device=DEV)
    elif k == "verify":
        n = _prefixes(c)
        cap = (max(n) + 8 + 7) // 8 * 8
        s["n"] = n
        s["q"] = g.normal((B, c["T"], Hq, d), dt)
        s["k"] = g.normal((B, Hkv, cap, d), dt)
        s["v"] = g.normal((B, Hkv, d, cap) if c["vt"] else (B, Hkv, cap, d), dt)
        s["kv"] = None if c["vt"] else mad.KV(s["k"], s["v"], n)
        s["out"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((B, c["T"], Hq), dtype=torch.float32, device=DEV)
    elif k == "greedy":
        T, V = c["T"], c["V"]
        s["logits"] = g.normal((B, T, V), dt)
        best = s["logits"].float().argmax(-1)[:, :T - 1].to(torch.int32)
        wrong = torch.randint(0, 4, best.shape, generator=g.g, device=DEV) == 0
        s["draft"] = torch.where(wrong, (best + 1) % V, best).to(torch.int32).contiguous()
        s["out"] = [torch.empty(B, dtype=torch.int32, device=DEV) for _ in range(2)]
    elif k == "stoch":
        T, V = c["T"], c["V"]
        z = g.normal((B, T, V), torch.float32)
        y = 0.8 * z[:, :T - 1] + 0.6 * g.normal((B, T - 1, V), torch.float32)
        s["p"], s["q"] = torch.softmax(z / 0.5, -1), torch.softmax(y / 0.5, -1).contiguous()
        s["draft"] = torch.multinomial(s["q"].view(-1, V), 1, generator=g.g).view(B, T - 1).to(torch.int32)
        s["uni"] = torch.rand((B, T), generator=g.g, device=DEV)
        s["out"] = [torch.empty(B, dtype=torch.int32, device=DEV) for _ in range(2)]
    elif k == "prefill":
        P = _prefixes(c)
        M = [_slots(p, c) for p in P]
        qc, sc = max(P), max(max(M), 1)
        s["P"], s["M"], s["c"] = P, M, c
        s["q"] = g.normal((B, qc, Hq, d), dt)
        s["qs"] = g.normal((B, sc, Hq, d), dt)
        s["raw"] = [g.normal((B, Hkv, qc, d), dt) for _ in range(2)]
        s["mem"] = [g.normal((B, Hkv, c["S"] + sc, d), dt) for _ in range(2)]
        s["raw_kv"] = mad.KV(*s["raw"], P)
        s["mem_kv"] = mad.KV(*s["mem"], [c["S"] + m if p > c["S"] else max(1, p) for p, m in zip(P, M)])
        s["out"] = [torch.zeros_like(s["q"]), torch.zeros((B, qc, Hq), dtype=torch.float32, device=DEV),
                    torch.zeros_like(s["qs"]), torch.zeros((B, sc, Hq), dtype=torch.float32, device=DEV)]
    elif k == "layer":
        s["w"] = _weights(c, g)
        s["lay"] = lay = MemoryLayout(c["S"], c["W"], c["r"], _ring_cap(c), c["S"] + c["p"] // c["r"] + c["u"] + 1, c["u"])
        s["ring"] = [g.normal((1, Hkv, lay.ring_cap, d), dt) for _ in range(2)]
        s["mem"] = [g.normal((1, Hkv, lay.mem_cap, d), dt) for _ in range(2)]
        s["x"] = g.normal((c["rows"], c["D"]), dt)
        s["p"] = c["p"]
        s["layer"] = DraftLayer(s["w"], c["D"], Hq, Hkv, d, c["F"], rope_base=ROPE_BASE, eps=EPS, device=DEV)
    else:
        R, D = c["rows"], c["D"]
        s["c"], s["w"] = c, _weights(c, g)
        s["x"], s["o"] = g.normal((R, D), dt), g.normal((R, Hq * d), dt)
        s["pos"] = [c["pos"] + 16 * i for i in range(R)]
        s["out"] = [torch.empty((R, n, d), dtype=dt, device=DEV) for n in (Hq, Hkv, Hkv)] + \
                   [torch.empty((R, n), dtype=dt, device=DEV) for n in (D, D, c["F"], D)]
    return s


def _weights(c, g):
    D, Hq, Hkv, d, F, bf = c["D"], c["Hq"], c["Hkv"], c["d"], c["F"], torch.bfloat16
    mk = lambda *shape: g.normal(shape, bf, std=0.02)
    return LayerWeights(gamma1=g.normal((D,), bf, 0.1, 1.0), w_qkv=mk((Hq + 2 * Hkv) * d, D), w_kv_g=mk(2 * Hkv * d, D),
                        w_o=mk(D, Hq * d), gamma2=g.normal((D,), bf, 0.1, 1.0), w_gate_up=mk(2 * F, D), w_down=mk(D, F))


# -------------------------------------------------------------------- run ----

def run(s):
    k = s["kind"]
    if k == "decode":
        out, lse = mad.draft_decode_attn(s["q"], s["mem_kv"], s["ring_kv"], s["kn"], s["vn"], s["out"], s["lse"])
        return {"out": out, "lse": lse, "ring": s["ring"]}
    if k == "boundary":
        mad.memory_update(s["x"], s["w"], s["pos"], s["upd_kv"], fire=s["fire"], rope_base=ROPE_BASE)
        out, lse = mad.draft_decode_attn(s["q"], s["mem_kv"], s["ring_kv"], s["kn"], s["vn"], s["out"], s["lse"])
        return {"out": out, "lse": lse, "ring": s["ring"], "mem": s["mem"]}
    if k == "step":
        mad.memory_update(s["x"], s["w"], s["pos"], s["upd_kv"], rope_base=ROPE_BASE)
        out, lse = mad.draft_step_attn(s["q"], s["mem_kv"], s["ring_kv"], s["kn"], s["vn"], s["modes"], s["out"], s["lse"])
        return {"out": out, "lse": lse, "ring": s["ring"], "mem": s["mem"]}
    if k == "verify":
        if s["kv"] is None:
            out, lse = mad.verify_attn_vt(s["q"], s["k"], s["v"], s["n"], s["out"], s["lse"])
        else:
            out, lse = mad.verify_attn(s["q"], s["kv"], s["out"], s["lse"])
        return {"out": out, "lse": lse}
    if k == "greedy":
        return list(mad.accept_greedy(s["logits"], s["draft"], *s["out"]))
    if k == "stoch":
        return list(mad.accept_stochastic(s["p"], s["q"], s["draft"], s["uni"], *s["out"]))
    if k == "prefill":
        c, o = s["c"], s["out"]
        return list(mad.memory_prefill_attn(s["q"], s["qs"], s["mem_kv"], s["raw_kv"], s["P"], c["S"], c["W"], c["r"],
                                            c["u"], *o))
    if k == "layer":
        y = s["layer"].step(s["x"], s["p"], s["lay"], *s["mem"], *s["ring"])
        return {"y": y, "ring": s["ring"], "mem": s["mem"]}
    c, w = s["c"], s["w"]
    q, kk, v, xn, h, a, y = s["out"]
    mad.rmsnorm_qkv_rope(s["x"], w.gamma1, w.w_qkv, s["pos"], c["Hq"], c["Hkv"], c["d"], q, kk, v, xn, eps=EPS,
                         rope_base=ROPE_BASE)
    mad.linear_residual(s["o"], w.w_o, s["x"], out=h)
    mad.rmsnorm_swiglu(h, w.gamma2, w.w_gate_up, out=a, eps=EPS)
    mad.linear_residual(a, w.w_down, h, out=y)
    return [q, kk, v, xn, h, a, y]


# ------------------------------------------------------------------- work ----

def _decode_keys(c, views):
    return sum(v[0] + v[1] + 1 for v in views)


def work(c):
    k, e = c["kind"], 4 if c.get("dtype") == "f32" else 2
    if k in ("greedy", "stoch"):
        if k == "greedy":
            return {"bytes": c["B"] * c["T"] * c["V"] * e, "flops": 0}
        return {"bytes": c["B"] * 2 * c["V"] * 4, "flops": c["B"] * 4 * c["V"]}
    Hq, Hkv, d = c["Hq"], c["Hkv"], c["d"]
    if k in ("decode", "boundary", "step"):
        if k == "step":
            rows, _ = _step_views(c)      # one sequence's rows share the keys: each is read once
            n_read = max(v[0] for v in rows) + c["W"] + c["r"] * c["u"]
            n, R = sum(v[0] + v[1] + (v[3] > 0) for v in rows), len(rows)
        else:
            n = _decode_keys(c, _views(c) if k == "decode" else _boundary_views(c)[0])
            n_read, R = n, c["B"]
        w = {"bytes": (n_read + R) * Hkv * d * 2 * e + 2 * R * Hq * d * e + R * Hq * 4, "flops": n * Hq * d * 4}
        if k != "decode":
            new = (sum(_fire(c)) if k == "boundary" else 1) * c["u"]
            w["bytes"] += (2 * Hkv * d * c["D"] + new * c["D"] + new * 2 * Hkv * d) * e
            w["flops"] += 2 * new * 2 * Hkv * d * c["D"]
        return w
    if k == "verify":
        n, T, B = sum(_prefixes(c)), c["T"], c["B"]
        return {"bytes": n * Hkv * d * 2 * e + 2 * B * T * Hq * d * e, "flops": n * T * Hq * d * 4}
    if k == "prefill":
        P, keys, rows = _prefixes(c), 0, 0
        for p in P:
            S, W, r = c["S"], c["W"], c["r"]
            for t in range(p):
                keys += min(S, t + 1) + _slots(t, c) + max(0, t + 1 - max(S, t - W + 1))
            m = _slots(p, c)
            keys += sum(S + i + min(W, i * r) for i in range(1, m + 1))
            rows += p + m
        return {"bytes": rows * (2 * Hq + 2 * Hkv) * d * 2 + rows * Hq * 4, "flops": keys * Hq * d * 4}
    D, F, R = c["D"], c["F"], c["rows"]
    weights = (Hq + 2 * Hkv) * d * D + Hq * d * D + 3 * F * D
    w = {"bytes": weights * 2, "flops": 2 * weights * R}
    if k == "layer":
        n = c["S"] + _slots(c["p"] + 1, c) + min(c["W"], c["p"] + 1 - c["S"])
        w["bytes"] += n * Hkv * d * 2 * 2 + (2 * Hkv * d * D * 2 if R > 1 else 0)
        w["flops"] += n * R * Hq * d * 4 + (2 * 2 * Hkv * d * D * (R - 1))
    return w


def tolerance(c):
    if c["kind"] in ("greedy", "stoch"):
        return "exact"
    # about four times what the results differ from 64 bits by (measured: fp32 sums 2.6e-7 to 4.8e-7; bf16 results
    # of fp32 sums 2.0e-3 to 2.3e-3; a layer, which rounds six intermediates to bf16 on the way, 3.3e-3)
    if c.get("dtype") == "f32":
        return {"rel": 2e-6}
    return {"rel": 1.3e-2 if c["kind"] in ("layer", "maps") else 9e-3}


# ------------------------------------------------------------------ exact ----

def _attend(q, K, V, scale):
    """q [Hkv, G, d], K and V [Hkv, n, d], 64 bits -> (out [Hkv, G, d], lse [Hkv, G])."""
    sc = torch.matmul(q, K.transpose(1, 2).contiguous()) * scale
    lse = torch.logsumexp(sc, -1)
    return torch.matmul(torch.exp(sc - lse[..., None]), V), lse


def _rope(x, pos):
    """x [..., n, H, d] rotated at pos [n] (rotate-half)."""
    d = x.shape[-1]
    th = ROPE_BASE ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    ang = torch.tensor(pos, dtype=torch.float64, device=x.device)[:, None, None] * th
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * torch.cos(ang) - b * torch.sin(ang), a * torch.sin(ang) + b * torch.cos(ang)], -1)


def _norm(x, gamma):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gamma.double()


def _update(x, w, pos, mem, rows, Hkv, d):
    """Slots of one sequence from x [n, D] into mem (a [Hkv, cap, d] pair, 64 bits) at `rows`."""
    y = torch.matmul(x, w.double().t().contiguous()).view(len(pos), 2, Hkv, d)
    mem[0][:, rows] = _rope(y[:, 0], pos).transpose(0, 1)
    mem[1][:, rows] = y[:, 1].transpose(0, 1)


def _rows(mem, ring, view, new):
    """The key (or value) list of a row: memory rows, ring rows, the new token."""
    m, n, st = view[:3]
    parts = [] if mem is None else [mem[:, :m].double()]
    idx = (st + torch.arange(n, device=ring.device)) % ring.shape[1]
    parts.append(ring[:, idx].double())
    if new is not None:
        parts.append(new[:, None].double())
    return torch.cat(parts, 1)


def exact(c, seed):
    k = c["kind"]
    s = prepare(c, seed)
    if k == "greedy":
        best = s["logits"].float().argmax(-1)
        miss = s["draft"] != best[:, :c["T"] - 1]
        a = torch.where(miss.any(1), miss.int().argmax(1), c["T"] - 1)
        return [a.to(torch.int32), best.gather(1, a[:, None])[:, 0].to(torch.int32)]
    if k == "stoch":
        return None
    Hq, Hkv, d = c["Hq"], c["Hkv"], c["d"]
    G, scale = Hq // Hkv, d ** -0.5
    if k in ("decode", "boundary", "step"):
        rows = s["q"].shape[0]
        ring = [t.double() for t in s["ring"]]
        mem = None if s["mem"] is None else [t.double() for t in s["mem"]]
        if k != "decode":
            for b in range(c["B"]):
                if k == "step" or s["fire"][b]:
                    at = s["upd_kv"].length[b]
                    _update(s["x"][b].double(), s["w"], s["pos"][b], [t[b] for t in mem],
                            slice(at, at + c["u"]), Hkv, d)
        out, lse = [], []
        for i in range(rows):
            b, v = (0 if k == "step" else i), s["views"][i]
            new = k != "step" or v[3] > 0
            K, V = (_rows(None if mem is None else mem[j][b], ring[j][b], v, s[("kn", "vn")[j]][i] if new else None)
                    for j in (0, 1))
            o, l = _attend(s["q"][i].double().view(Hkv, G, d), K, V, scale)
            out.append(o.reshape(Hq, d))
            lse.append(l.reshape(Hq))
        for i in range(rows):
            if k != "step" or s["views"][i][3] == 2:
                v, b = s["views"][i], 0 if k == "step" else i
                at = (v[2] + v[1]) % ring[0].shape[2]
                ring[0][b][:, at], ring[1][b][:, at] = s["kn"][i].double(), s["vn"][i].double()
        got = {"out": torch.stack(out), "lse": torch.stack(lse), "ring": ring}
        return got if k == "decode" else dict(got, mem=mem)
    if k == "verify":
        T, out, lse = c["T"], [], []
        for b, n in enumerate(s["n"]):
            K = s["k"][b, :, :n].double()
            V = (s["v"][b, :, :, :n].transpose(1, 2) if c["vt"] else s["v"][b, :, :n]).double().contiguous()
            q = s["q"][b].double().view(T, Hkv, G, d).transpose(0, 1).reshape(Hkv, T * G, d)
            sc = torch.matmul(q, K.transpose(1, 2).contiguous()) * scale
            lim = n - T + torch.arange(T, device=DEV).repeat_interleave(G)
            sc.masked_fill_(torch.arange(n, device=DEV)[None, :] > lim[:, None], -math.inf)
            l = torch.logsumexp(sc, -1)
            o = torch.matmul(torch.exp(sc - l[..., None]), V)
            out.append(o.view(Hkv, T, G, d).transpose(0, 1).reshape(T, Hq, d))
            lse.append(l.view(Hkv, T, G).transpose(0, 1).reshape(T, Hq))
        return {"out": torch.stack(out), "lse": torch.stack(lse)}
    if k == "prefill":
        return _exact_prefill(c, s)
    if k == "layer":
        return _exact_layer(c, s)
    w, x = s["w"], s["x"].double()
    xn = _norm(x, w.gamma1)
    q, kk, v = _qkv(c, w, xn, s["pos"])
    h = x + torch.matmul(s["o"].double(), w.w_o.double().t().contiguous())
    a, y = _mlp(c, w, h)
    return [q, kk, v, xn, h, a, y]


def _qkv(c, w, xn, pos):
    Hq, Hkv, d = c["Hq"], c["Hkv"], c["d"]
    y = torch.matmul(xn, w.w_qkv.double().t().contiguous()).view(-1, Hq + 2 * Hkv, d)
    return _rope(y[:, :Hq], pos), _rope(y[:, Hq:Hq + Hkv], pos), y[:, Hq + Hkv:]


def _mlp(c, w, h):
    gu = torch.matmul(_norm(h, w.gamma2), w.w_gate_up.double().t().contiguous())
    a = torch.nn.functional.silu(gu[:, :c["F"]]) * gu[:, c["F"]:]
    return a, h + torch.matmul(a, w.w_down.double().t().contiguous())


def _exact_prefill(c, s):
    Hq, Hkv, d, S, W, r = c["Hq"], c["Hkv"], c["d"], c["S"], c["W"], c["r"]
    G, scale, QB = Hq // Hkv, c["d"] ** -0.5, 256
    outs = [torch.zeros(t.shape, dtype=torch.float64, device=DEV) for t in s["out"]]

    def block(q, K, V, Kr, Vr, mlim, lo, hi, base):
        # q [n, Hq, d]; memory rows below mlim [n], raw rows [lo, hi) of rows base ..
        n = q.shape[0]
        qq = q.double().view(n, Hkv, G, d).permute(1, 0, 2, 3).reshape(Hkv, n * G, d)
        keys, vals = torch.cat([K, Kr], 1), torch.cat([V, Vr], 1)
        at = torch.arange(K.shape[1], device=DEV)
        ar = base + torch.arange(Kr.shape[1], device=DEV)
        ok = torch.cat([at[None] < mlim[:, None], (ar[None] >= lo[:, None]) & (ar[None] < hi[:, None])], 1)
        sc = torch.matmul(qq, keys.transpose(1, 2).contiguous()) * scale
        sc.masked_fill_(~ok.repeat_interleave(G, 0), -math.inf)
        l = torch.logsumexp(sc, -1)
        o = torch.matmul(torch.exp(sc - l[..., None]), vals)
        return (o.view(Hkv, n, G, d).permute(1, 0, 2, 3).reshape(n, Hq, d), l.view(Hkv, n, G).permute(1, 0, 2).reshape(n, Hq))

    for b, (P, M) in enumerate(zip(s["P"], s["M"])):
        mk, mv = (t[b].double() for t in s["mem"])
        rk, rv = (t[b].double() for t in s["raw"])
        for kind, nq in ((0, P), (1, M)):
            for q0 in range(0, nq, QB):
                q1 = min(nq, q0 + QB)
                if kind == 0:
                    t = torch.arange(q0, q1, device=DEV)
                    made = torch.clamp(t - S, min=0) // (r * c["u"]) * c["u"]
                    mlim = torch.where(t < S, t + 1, S + made)
                    lo = torch.clamp(t - W + 1, min=S)
                    hi = torch.where(t < S, lo, t + 1)
                else:
                    m = torch.arange(q0 + 1, q1 + 1, device=DEV)
                    mlim, hi = S + m, S + m * r
                    lo = torch.clamp(hi - W, min=S)
                m1, r0, r1 = int(mlim.max()), int(lo.min()), max(int(hi.max()), int(lo.min()))
                o, l = block((s["q"], s["qs"])[kind][b, q0:q1], mk[:, :m1], mv[:, :m1], rk[:, r0:r1], rv[:, r0:r1],
                             mlim, lo, hi, r0)
                outs[2 * kind][b, q0:q1], outs[2 * kind + 1][b, q0:q1] = o, l
    return outs


def _exact_layer(c, s):
    Hq, Hkv, d, R, p = c["Hq"], c["Hkv"], c["d"], c["rows"], c["p"]
    w, x = s["w"], s["x"].double()
    ring, mem = [t.double() for t in s["ring"]], [t.double() for t in s["mem"]]
    before = _slots(p, c)
    pos = [p] + [c["S"] + (before + 1 + i) * c["r"] for i in range(R - 1)]
    xn = _norm(x, w.gamma1)
    q, kk, v = _qkv(c, w, xn, pos)
    cap = ring[0].shape[2]
    n, st = _win(c, p - c["W"] + 1, p, cap)
    rows = [(c["S"] + before, n, st, True)]
    if R > 1:
        _update(xn[1:], w.w_kv_g, pos[1:], [t[0] for t in mem], slice(c["S"] + before, c["S"] + before + R - 1), Hkv, d)
        for i in range(1, R):
            wn, ws = _win(c, pos[i] - c["W"], pos[i], cap)
            last = pos[i] - 1 == p
            rows.append((c["S"] + before + i, wn - 1 if last else wn, ws, last))
    o = []
    for i, view in enumerate(rows):
        K, V = (_rows(mem[j][0], ring[j][0], view, (kk, v)[j][0] if view[3] else None) for j in (0, 1))
        o.append(_attend(q[i].view(Hkv, Hq // Hkv, d), K, V, d ** -0.5)[0].reshape(Hq * d))
    at = (st + n) % cap
    ring[0][0][:, at], ring[1][0][:, at] = kk[0], v[0]
    h = x + torch.matmul(torch.stack(o), w.w_o.double().t().contiguous())
    return {"y": _mlp(c, w, h)[1], "ring": ring, "mem": mem}
