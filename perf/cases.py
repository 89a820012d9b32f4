"""What this framework is timed on: decode attention over a four-tier KV cache, through the public binding.

Four kinds of pass, all on synthetic reasoning-shaped caches (standard normal keys, values and queries; one key element
carries a per-position importance z ~ N(0, 1) and the matching query element is sqrt(head_dim), so that a position's
average attention weight is log-normal over the positions, the long tail of the paper's Sec. 2.1):

  attend   some decode steps' attention as a model calls it: one `attend_and_score` per layer, in layer order, over a
           cache whose rows already lie in their tiers (two score-driven re-tierings behind them, so the slots of list
           neighbours are scattered as in a running request); then the importance scores are read once.
  chunk    the same for several query tokens per sequence at once (`attend_and_score_chunk`: drafted tokens, a short
           prompt tail).
  retier   one stationary re-tiering period: the importance scores are set, `classify` + `migrate` move the rows whose
           band changed (T1 rows over the host link, lazily, beside the attention that follows), then `steps` steps of
           per-layer attention; scores and tiers are read.  The two score arrays take turns, so every pass moves rows.
  request  a whole request: create the cache, append the context of every layer, `steps` whole `decode_step`s with a
           re-tiering after every `delta` of them, read scores and tiers, close.

Shapes, policies and formats are those of this repository's benchmark configurations (tkv_synth.py, bench.py), with the
layers cut where one layer more adds nothing but time; contexts are odd where a running request's would be.
"""
import math

import numpy as np
import torch

import paper_2605_09490_amd as tkv

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
BASE = dict(kind="attend", layers=1, batch=1, q_heads=8, kv_heads=2, dim=64, dtype="bf16", out="f32", t2="int8_row", mode="lazy",
            scorer="attention", context=512, window=128, f0=500_000, f1=350_000, f2=100_000, f3=50_000, steps=1, n_q=1, delta=0)
MIX_TINY = dict(f0=500_000, f1=300_000, f2=150_000, f3=50_000)
MIX_7B = dict(f0=500_000, f1=350_000, f2=100_000, f3=50_000)
MIX_14B = dict(f0=300_000, f1=520_000, f2=150_000, f3=30_000)
MIX_32B = dict(f0=300_000, f1=500_000, f2=100_000, f3=100_000)
MIX_PROD = dict(f0=300_000, f1=470_000, f2=200_000, f3=30_000)
MIX_HBM = dict(f0=820_000, f1=0, f2=150_000, f3=30_000)     # the 14B policy with T1 folded into T0: no host link in it


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    b7 = dict(q_heads=28, kv_heads=4, dim=128, **MIX_7B)
    b14 = dict(batch=8, q_heads=40, kv_heads=8, dim=128)
    return [
        # the smallest calls: one sequence, one small binary32 layer, 32 decode steps; launches and latency are all there is
        _case("tiny_f32", dtype="f32", context=512, window=32, steps=32, **MIX_TINY),
        # one user's request on the 7B shape, at the paper's mean chain length: few rows per layer, 28 layers
        _case("solo_7b", layers=28, context=1422, steps=4, **b7),
        # the 7B benchmark shape: a small batch, short lists, groups of 7 heads
        _case("7b", layers=28, batch=8, context=2081, steps=2, **b7),
        # the 14B benchmark shape (the headline): 123 MB per layer call
        _case("14b", layers=8, context=4133, steps=4, **b14, **MIX_14B),
        # the 32B benchmark shape: half the batch, twice the context; binary16 cache and output
        _case("32b_f16", layers=8, batch=4, q_heads=40, kv_heads=8, dim=128, dtype="f16", out="f16", context=8201, steps=4, **MIX_32B),
        # the production batch: 64 sequences of 16384 tokens, int4 T2, 1.8 GB per layer call (the largest)
        _case("prod_int4", batch=64, q_heads=28, kv_heads=4, dim=128, t2="int4_g32", context=16384, steps=16, **MIX_PROD),
        # four drafted tokens per sequence verified at once on the 14B shape
        _case("chunk4_14b", kind="chunk", layers=8, context=4133, steps=2, n_q=4, **b14, **MIX_14B),
        # a longer draft of odd length on the 7B shape, binary16 cache, int4 T2
        _case("chunk13_7b_f16", kind="chunk", layers=8, batch=8, dtype="f16", t2="int4_g32", context=2081, steps=2, n_q=13, **b7),
        # one re-tiering period of 16 steps on the 14B shape, rows moving between all tiers
        _case("retier_14b", kind="retier", layers=8, context=4112, steps=16, **b14, **MIX_14B),
        # one user's whole request, T1 offloaded over the host link
        _case("request_solo_7b", kind="request", layers=28, context=1422, steps=32, delta=16, **b7),
        # the 7B benchmark configuration, whole
        _case("request_7b", kind="request", layers=28, batch=8, context=2048, steps=64, delta=16, **b7),
        # the 14B benchmark configuration at full depth with everything kept in HBM
        _case("request_14b", kind="request", layers=48, context=4096, steps=32, delta=16, **b14, **MIX_HBM),
    ]


def _row_bytes(c):
    es = 4 if c["dtype"] == "f32" else 2
    full = 2 * c["dim"] * es
    t2 = 2 * (c["dim"] + 4) if c["t2"] == "int8_row" else 2 * (c["dim"] // 2 + c["dim"] // 16)
    return es, full, t2


def _mean_row_bytes(c):
    _, full, t2 = _row_bytes(c)
    return ((c["f0"] + c["f1"]) * full + c["f2"] * t2) / 1e6


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["attend", "attend", "attend", "chunk", "retier", "request"])
    heads = rng.choice([(8, 2), (28, 4), (28, 4), (40, 8), (40, 8), (10, 2), (8, 8), (16, 4), (64, 8), (12, 2)])
    c = dict(BASE, kind=kind, q_heads=heads[0], kv_heads=heads[1], dim=rng.choice([64, 128, 128, 128]),
             dtype=rng.choice(["bf16", "bf16", "bf16", "f16", "f32"]), out=rng.choice(["f32", "f32", "bf16"]),
             t2=rng.choice(["int8_row", "int8_row", "int4_g32"]), window=rng.choice([32, 128]), mode=rng.choice(["lazy", "lazy", "wait"]))
    c.update(rng.choice([MIX_TINY, MIX_7B, MIX_14B, MIX_32B, MIX_PROD]))
    if kind == "request":
        c.update(layers=rng.randint(1, 28), batch=log_int(1, 16), context=log_int(300, 6000), delta=16, steps=rng.choice([16, 32, 48]),
                 scorer=rng.choice(["attention", "attention", "vatp"]))
        most = 1.0e9          # bytes of cache read by one step
    elif kind == "retier":
        c.update(layers=rng.randint(2, 12), batch=log_int(1, 16), context=log_int(500, 8000), steps=16)
        most = 1.0e9
    else:
        c.update(layers=rng.randint(1, 28), batch=log_int(1, 64), context=log_int(300, 16384))
        most = 1.7e9
    rows = _mean_row_bytes(c) * c["kv_heads"] * c["batch"]
    c["context"] = max(257, min(c["context"], int(most / rows)))
    c["layers"] = max(1, min(c["layers"], int(most / (rows * c["context"]))))
    if kind in ("attend", "chunk"):
        if kind == "chunk":
            c["n_q"] = rng.randint(2, 20)
            c["mode"] = "lazy"
        passes = 2.0e9 / (rows * c["context"] * c["layers"]) / (c["n_q"] if c["dtype"] == "f32" else 1)
        c["steps"] = max(1, min(32, int(passes), 600 // c["layers"]))
    return c


# ---- inputs ------------------------------------------------------------------------------------------------------
def _generator(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + tag * 7919 + 12345) & 0x7FFFFFFFFFFFFFFF)
    return g


class _Inputs:
    """Everything a pass is given, drawn from the seed."""

    def __init__(self, c, seed):
        self.c, self.seed = c, seed
        self.dt = DTYPES[c["dtype"]]
        extra = c["n_q"] if c["kind"] == "chunk" else c["steps"] if c["kind"] == "request" else 0
        self.n0, self.total = c["context"], c["context"] + extra
        g = _generator(seed, 1)
        self.z = torch.randn((c["batch"], self.total), generator=g, device="cuda")
        # importance as earlier steps of a request would have left it: the long tail, twice, 25 % of its logarithm redrawn
        self.s = []
        for _ in range(2):
            s = torch.exp(self.z + 0.25 * torch.randn(self.z.shape, generator=g, device="cuda"))
            s[:, c["context"]:] = 0.0
            self.s.append((s * (16.0 / s.sum(1, keepdim=True))).float().contiguous())

    def rows(self, layer, lo, hi, tag):
        """Keys and values [B, hi - lo, Hkv, D] of positions lo .. hi - 1."""
        c = self.c
        g = _generator(self.seed, 1000 + 64 * layer + tag)
        shape = (c["batch"], hi - lo, c["kv_heads"], c["dim"])
        k = torch.randn(shape, generator=g, device="cuda", dtype=self.dt)
        v = torch.randn(shape, generator=g, device="cuda", dtype=self.dt)
        k[..., 0] = self.z[:, lo:hi, None].to(self.dt)
        return k, v

    def queries(self):
        """[steps, L, B, (n_q,) Hq, D]"""
        c = self.c
        shape = [c["steps"], c["layers"], c["batch"], c["q_heads"], c["dim"]]
        if c["kind"] == "chunk":
            shape.insert(3, c["n_q"])
        q = torch.randn(shape, generator=_generator(self.seed, 2), device="cuda", dtype=self.dt)
        q[..., 0] = math.sqrt(c["dim"])
        return q

    def new_rows(self):
        """A request's generated rows, [steps, L, B, 1, Hkv, D]."""
        c = self.c
        g = _generator(self.seed, 3)
        shape = (c["steps"], c["layers"], c["batch"], 1, c["kv_heads"], c["dim"])
        k = torch.randn(shape, generator=g, device="cuda", dtype=self.dt)
        v = torch.randn(shape, generator=g, device="cuda", dtype=self.dt)
        k[..., 0] = self.z[:, self.n0:].t()[:, None, :, None, None].to(self.dt)
        return k, v


def _policy(c):
    return (c["f0"], c["f1"], c["f2"], c["f3"])


def _cache(c, max_tokens):
    """A cache with pools sized for the policy's shares (and the rows that enter before others leave)."""
    n = max_tokens
    share = lambda ppm, over: min(n, int(over * ppm * n) // 1_000_000 + 64)
    return tkv.TieredKV(c["layers"], c["batch"], c["q_heads"], c["kv_heads"], c["dim"], n, kv_dtype=c["dtype"], t2_format=c["t2"],
                        out_dtype=c["out"], k_sink=4, k_window=c["window"], prefetch_mode=c["mode"], scorer=c["scorer"],
                        staging_rows=share(c["f1"], 1.5), t2_rows=share(c["f2"], 2.5),
                        host_rows=min(c["batch"] * n, int(1.6 * c["f1"] * c["batch"] * n) // 1_000_000 + 64 * c["batch"]))


def prepare(case, seed):
    c = case
    x = _Inputs(c, seed)
    st = {"case": c, "max_tokens": x.total}
    q = x.queries()
    out = torch.zeros(q.shape, dtype=DTYPES[c["out"]], device="cuda")
    if c["kind"] == "request":
        k, v = zip(*[x.rows(l, 0, x.n0, 0) for l in range(c["layers"])])
        kn, vn = x.new_rows()
        st.update(k=k, v=v, kn=kn, vn=vn, q=q, out=out)
        return st
    kv = _cache(c, x.total)
    for l in range(c["layers"]):
        kv.append(l, *x.rows(l, 0, x.n0, 0))
    scores = [s.cpu().numpy() for s in x.s]
    for s in (scores[1],) if c["kind"] == "retier" else scores:
        kv.set_scores(s)
        kv.classify(_policy(c))
        kv.migrate()
    kv.wait_prefetch()
    if c["kind"] == "chunk":
        for l in range(c["layers"]):
            kv.append(l, *x.rows(l, x.n0, x.total, 1))
    # the buffers of every layer call, as a model's layers hold them
    calls = [(l, q[s, l], out[s, l]) for s in range(c["steps"]) for l in range(c["layers"])]
    st.update(kv=kv, calls=calls, q=q, out=out, scores=scores, turn=0)
    return st


def run(st):
    c = st["case"]
    if c["kind"] == "request":
        kv = _cache(c, st["max_tokens"])
        for l in range(c["layers"]):
            kv.append(l, st["k"][l], st["v"][l])
        for s in range(c["steps"]):
            kv.decode_step(st["kn"][s], st["vn"][s], st["q"][s], st["out"][s])
            if (s + 1) % c["delta"] == 0:
                kv.classify(_policy(c))
                kv.migrate()
        res = {"out": st["out"], "scores": kv.get_scores(), "tiers": kv.get_tiers()}
        kv.close()
        return res
    kv = st["kv"]
    if c["kind"] == "chunk":
        for l, q, o in st["calls"]:
            kv.attend_and_score_chunk(l, q, o)
        return {"out": st["out"], "scores": kv.get_scores()}
    if c["kind"] == "retier":
        kv.set_scores(st["scores"][st["turn"]])
        st["turn"] ^= 1
        kv.classify(_policy(c))
        kv.migrate()
    for l, q, o in st["calls"]:
        kv.attend_and_score(l, q, o)
    res = {"out": st["out"], "scores": kv.get_scores()}
    if c["kind"] == "retier":
        res["tiers"] = kv.get_tiers()
    return res


def work(case):
    """One pass: every row that is attended read once per layer call, queries read, outputs written, scores updated; a
    request's context and new rows read and stored, a re-tiering's moved rows (about a tenth of the rows) not counted."""
    c = case
    es, full, t2 = _row_bytes(c)
    oes = 4 if c["out"] == "f32" else 2
    total = flops = 0.0
    for s in range(c["steps"]):
        n = c["context"] + (s + 1 if c["kind"] == "request" else c["n_q"] if c["kind"] == "chunk" else 0)
        tiered = c["kind"] != "request" or s >= c["delta"]
        u = max(0, c["context"] - 4 - c["window"]) if tiered else 0
        n2, n3 = u * c["f2"] // 1_000_000, u * c["f3"] // 1_000_000
        n1 = n - n2 - n3
        heads = c["batch"] * c["n_q"] * c["q_heads"] * c["dim"]
        total += c["layers"] * (c["batch"] * c["kv_heads"] * (n1 * full + n2 * t2) + heads * (es + oes) + c["batch"] * (n - n3) * 8)
        flops += c["layers"] * 4.0 * heads * (n - n3)
    if c["kind"] == "request":
        total += 2.0 * c["layers"] * c["batch"] * c["kv_heads"] * (c["context"] + c["steps"]) * full
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """Outputs and scores are binary32 sums over inputs that are exact in 16 bits (binary32 in tiny): another order of the
    same sums is a few 1e-7 off, and a 16-bit output adds its own rounding where a value falls on the other side.  A
    request's ranking may turn round for neighbours whose scores agree to the last bits: one row then sits in another tier."""
    out16 = case["out"] != "f32"
    if case["kind"] == "request":
        return {"rel": 2e-3, "max": 0.2, "differ": 1e-3}
    return {"rel": 1e-3 if case["out"] == "bf16" else 2e-4 if out16 else 3e-6, "max": 2e-2 if out16 else 1e-4, "differ": 1e-4}


# ---- the same in 64 bits ---------------------------------------------------------------------------------------------
def _decoded(x, t2):
    """Rows [..., D] as T2 holds them: the codes of the stated binary32 encoder, times their scale in 64 bits."""
    x = x.float()
    if t2 == "int8_row":
        top, a = 127.0, x.abs().amax(-1, keepdim=True)
        scale = a / torch.full_like(a, top)          # a true division: by a plain number it would be a product with the reciprocal
        y = x
    else:
        y = x.reshape(*x.shape[:-1], x.shape[-1] // 32, 32)
        top, a = 7.0, y.abs().amax(-1, keepdim=True)
        scale = (a / torch.full_like(a, top)).half().float()
    code = torch.where(scale > 0, torch.round(y / torch.where(scale > 0, scale, torch.ones_like(scale))).clamp(-top, top), torch.zeros_like(y))
    return (code.double() * scale.double()).reshape(x.shape)


def _plan(c, score32, tier, n):
    """Tiers of positions 0 .. n-1: evicted first, then by score, then by position; the bands' floors of the policy."""
    lo, hi = 4, n - c["window"]
    new = torch.zeros_like(tier)
    if hi <= lo:
        return new
    m = hi - lo
    n3, n2, n0 = m * c["f3"] // 1_000_000, m * c["f2"] // 1_000_000, m * c["f0"] // 1_000_000
    for b in range(tier.shape[0]):
        key = torch.where(tier[b, lo:hi] == 3, torch.full_like(score32[b, lo:hi], -math.inf), score32[b, lo:hi])
        order = torch.sort(key, stable=True).indices + lo
        evicted = int((tier[b, lo:hi] == 3).sum())
        c3, c2, c0 = n3, n2, n0
        extra = max(0, evicted - n3)
        c3 += extra
        t = min(extra, c2); c2 -= t; extra -= t
        c1 = m - n3 - n2 - n0
        t = min(extra, c1); c1 -= t; extra -= t
        new[b, order[:c3]] = 3
        new[b, order[c3:c3 + c2]] = 2
        new[b, order[c3 + c2:c3 + c2 + c1]] = 1
    return new


def _attend64(c, q, k, v, tier, first, per_call):
    """q [T, B, Hq, D]; k, v [B, n, Hkv, D] stored rows; query j sees positions < first + j (all of them where per_call).
    Returns out [T, B, Hq, D] in 64 bits and the weights' sums over heads [T, B, n]."""
    T, B, Hq, D = q.shape
    n, Hkv = k.shape[1], k.shape[2]
    G = Hq // Hkv
    outs, sums = [], []
    for b in range(B):
        t2 = (tier[b] == 2)[:, None, None]
        kb = torch.where(t2, _decoded(k[b], c["t2"]), k[b].double()).permute(1, 2, 0).contiguous()       # [Hkv, D, n]
        vb = torch.where(t2, _decoded(v[b], c["t2"]), v[b].double()).permute(1, 0, 2).contiguous()       # [Hkv, n, D]
        qb = q[:, b].double().reshape(T, Hkv, G, D).permute(1, 0, 2, 3).reshape(Hkv, T * G, D).contiguous()
        x = torch.matmul(qb, kb) / math.sqrt(D)
        x.masked_fill_((tier[b] == 3)[None, None, :], -math.inf)
        if not per_call:
            last = (first + torch.arange(T, device="cuda")).repeat_interleave(G)
            x.masked_fill_((torch.arange(n, device="cuda")[None, :] >= last[:, None])[None], -math.inf)
        p = torch.softmax(x, -1)
        o = torch.matmul(p, vb).reshape(Hkv, T, G, D).permute(1, 0, 2, 3).reshape(T, Hq, D)
        w = p.reshape(Hkv, T, G, n).sum(2)                                                                # [Hkv, T, n]
        if c["scorer"] == "vatp":
            w = w * v[b].double().norm(dim=-1).t()[:, None, :]
        outs.append(o)
        sums.append(w.sum(0))
    return torch.stack(outs, 1), torch.stack(sums, 1)


def _round_rows(x, moved, dt, t2):
    """Rows that leave T2 are stored as code * scale (binary32), rounded to the cache's type."""
    return torch.where(moved[:, :, None, None], _decoded(x, t2).float().to(dt), x)


def exact(case, seed):
    c = case
    es, full, _ = _row_bytes(c)
    cost = c["layers"] * c["batch"] * c["kv_heads"] * c["context"] * c["dim"]
    if cost * (3 if c["kind"] == "request" else 1) > 6.0e9 or c["steps"] * c["n_q"] * c["batch"] * c["layers"] > 40_000:
        return None
    x = _Inputs(c, seed)
    B, dt, N = c["batch"], DTYPES[c["dtype"]], x.total
    scale = 1.0 / (c["layers"] * c["q_heads"])
    q = x.queries()
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    tier = torch.zeros((B, N), dtype=torch.uint8, device="cuda")
    if c["kind"] == "request":
        if c["scorer"] != "attention":
            return None
        ks, vs = zip(*[x.rows(l, 0, x.n0, 0) for l in range(c["layers"])])
        kn, vn = x.new_rows()
        ks = [torch.cat([ks[l], kn[:, l, :, 0].transpose(0, 1)], 1) for l in range(c["layers"])]
        vs = [torch.cat([vs[l], vn[:, l, :, 0].transpose(0, 1)], 1) for l in range(c["layers"])]
        score = torch.zeros((B, N), dtype=torch.float64, device="cuda")
        for s0 in range(0, c["steps"], c["delta"]):
            m = min(c["delta"], c["steps"] - s0)
            n = x.n0 + s0 + m
            for l in range(c["layers"]):
                o, w = _attend64(c, q[s0:s0 + m, l], ks[l][:, :n], vs[l][:, :n], tier[:, :n], x.n0 + s0 + 1, False)
                out[s0:s0 + m, l] = o
                score[:, :n] += scale * w.sum(0)
            if m == c["delta"]:
                new = tier.clone()
                new[:, :n] = _plan(c, score[:, :n].float(), tier[:, :n], n)
                moved = (tier == 2) & (new != 2)
                for l in range(c["layers"]):
                    ks[l] = _round_rows(ks[l], moved, dt, c["t2"])
                    vs[l] = _round_rows(vs[l], moved, dt, c["t2"])
                tier = new
        return {"out": out, "scores": score.cpu().numpy(), "tiers": None}
    n0 = x.n0
    t1 = tier.clone()
    t1[:, :n0] = _plan(c, x.s[1 if c["kind"] == "retier" else 0][:, :n0], tier[:, :n0], n0)
    t2 = t1.clone()
    t2[:, :n0] = _plan(c, x.s[0 if c["kind"] == "retier" else 1][:, :n0], t1[:, :n0], n0)
    moved = (t1 == 2) & (t2 != 2)
    score = x.s[0 if c["kind"] == "retier" else 1].double().clone()
    for l in range(c["layers"]):
        k, v = x.rows(l, 0, n0, 0)
        if c["kind"] == "chunk":
            kn, vn = x.rows(l, n0, N, 1)
            k, v = torch.cat([k, kn], 1), torch.cat([v, vn], 1)
        k, v = _round_rows(k, moved, dt, c["t2"]), _round_rows(v, moved, dt, c["t2"])
        if c["kind"] == "chunk":
            for s in range(c["steps"]):
                o, w = _attend64(c, q[s, l].transpose(0, 1), k, v, t2, n0 + 1, False)
                out[s, l] = o.transpose(0, 1)
                score += scale * w.sum(0)
        else:
            o, w = _attend64(c, q[:, l], k, v, t2, n0, True)
            out[:, l] = o
            score += scale * w.sum(0)
    res = {"out": out, "scores": score.cpu().numpy()}
    if c["kind"] == "retier":
        res["tiers"] = None
    return res
