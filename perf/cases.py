"""Timed cases of the H2O attention path, called through the public Python binding.

Every case is one pass of something a program that generates text with an H2O
cache does over and over: a generation step of one layer, the prompt phase of one
layer (with or without the prompt's attention output, in one piece or in chunks)
followed by the first generated token, the compression of a prompt whose scores
are known, and one whole short generation.  Shapes are those of the workload
table in synth.py (OPT-6.7B and OPT-30B shaped layers, the 4096-token prompt, the
small binary32 layer), plus single sequences, odd lengths and long budgets in
between.

A case is a dict of plain values; `prepare` makes its inputs and its cache on the
GPU, `run` is one pass, `exact` the same outputs from plain torch in float64.
"""
import math

import torch

from paper_2306_14048_amd import binding as h2o

DEV = "cuda"
DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
TOKENS = 8          # distinct new tokens a stepping program cycles through here


def _case(name, kind, batch, heads, d, dtype, n, heavy, recent, **more):
    c = dict(kind=kind, batch=batch, heads=heads, d=d, dtype=dtype, n=n, heavy=heavy, recent=recent,
             sigma=1.0, rank=0, kv_bits=0, chunk=0, steps=1)
    c.update(more)
    if name:
        c["name"] = name
    return c


def _split(k):
    return (k + 1) // 2, k - (k + 1) // 2


def listed():
    return [
        # -- generation steps of one layer (the bulk of a program's calls) --------------
        # the smallest call: one short sequence on a small binary32 layer; all latency
        _case("step small f32", "step", 1, 8, 64, "f32", 64, 32, 32, sigma=0.75),
        # one sequence of an OPT-6.7B layer, 2048-token prompt at 20 %: interactive serving
        _case("step one sequence f16", "step", 1, 32, 128, "f16", 410, 205, 205),
        # the same layer at batch 16: the benchmark's step
        _case("step batch f16", "step", 16, 32, 128, "f16", 410, 205, 205),
        # an OPT-30B layer at batch 64, 1024-token prompts at 20 %: throughput serving
        _case("step wide batch f16", "step", 64, 56, 128, "f16", 205, 103, 102),
        # two sequences with 16 k of context at 20 %: few heads, a long budget
        _case("step long budget bf16", "step", 2, 32, 128, "bf16", 3277, 1639, 1638),
        # the batch-16 step on the 4-bit cache
        _case("step batch 4-bit f16", "step", 16, 32, 128, "f16", 410, 205, 205, kv_bits=4),
        # -- prompt phase + first generated token of one layer ---------------------------
        # scores only (the program has its own attention): batch 16, 2048 tokens
        _case("prompt scores batch f16", "scores", 16, 32, 128, "f16", 2048, 205, 205),
        # with the attention output: 4 prompts of 4096 tokens
        _case("prompt attention bf16", "attention", 4, 32, 128, "bf16", 4096, 410, 409),
        # one prompt of an odd length: time to the first token
        _case("prompt one sequence f16", "attention", 1, 32, 128, "f16", 1531, 153, 153),
        # 4 prompts of 4096 tokens fed in chunks of 1024, with the attention output
        _case("prompt chunked bf16", "chunked", 4, 32, 128, "bf16", 4096, 410, 409, chunk=1024),
        # -- the rest ----------------------------------------------------------------------
        # compression with scores from elsewhere: one 16 k prompt, 20 % kept
        _case("compress one long f16", "compress", 1, 32, 128, "f16", 16384, 1639, 1638),
        # a whole short generation: 256 prompt tokens and 64 steps on the small layer
        _case("generation small f32", "generation", 1, 8, 64, "f32", 256, 32, 32, sigma=0.75, steps=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step4", "scores", "attention", "chunked", "compress",
                       "generation"])
    heads = rng.choice([8, 12, 16, 32, 32, 56])
    d = rng.choice([64, 128, 128])
    dtype = rng.choice(["f16", "bf16", "f16", "bf16", "f32"])
    rank = rng.choice([0, 0, 0, 1])
    if kind in ("step", "step4"):
        # 8 .. 3584 heads, budgets 48 .. 4096 (4-bit: 2048), at most the bytes of the widest listed step
        k = _log_int(rng, 48, 2048 if kind == "step4" else 4096)
        row = 2 * d * (4 if dtype == "f32" else 2)
        most = max(1, min(64, int(376e6 / (heads * k * row))))
        batch = _log_int(rng, 1, most)
        heavy, recent = _split(k)
        return _case(None, "step", batch, heads, d, dtype, k, heavy, recent, rank=rank,
                     kv_bits=4 if kind == "step4" else 0)
    if kind == "compress":
        n = _log_int(rng, 256, 16384)
        batch = _log_int(rng, 1, max(1, min(16, int(2.1e6 / (heads * n)))))
        heavy, recent = _split(max(16, int(n * rng.uniform(0.05, 0.25))))
        return _case(None, kind, batch, heads, d, dtype, n, heavy, recent, rank=rank)
    if kind == "generation":
        n = _log_int(rng, 64, 512)
        heavy, recent = _split(max(16, int(n * rng.uniform(0.1, 0.3))))
        return _case(None, kind, rng.choice([1, 2, 4]), heads, d, dtype, n, heavy, recent,
                     sigma=0.75, steps=rng.choice([16, 32, 64]))
    if kind != "scores" and dtype == "f32":
        dtype = "f16"                                   # 16-bit element types only
    n = _log_int(rng, 100, 6000 if dtype != "f32" else 1500)
    most = max(1, min(32, int(2.1e9 / (heads * n * n))))
    batch = _log_int(rng, 1, most)
    heavy, recent = _split(max(16, min(4096, int(n * rng.uniform(0.05, 0.25)))))
    chunk = min(n, rng.choice([256, 512, 1000, 1024, 2048])) if kind == "chunked" else 0
    return _case(None, kind, batch, heads, d, dtype, n, heavy, recent, rank=rank, chunk=chunk)


# ---- inputs -----------------------------------------------------------------------------
def _randn(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)


def _inputs(c, seed):
    """Q, K, V of the prompt [B, Hh, n, d], q, k, v of the new tokens [T, B, Hh, d] and (step and
    compress) a score per prompt token.  Values as in synth.py: N(0, 1), key rows scaled by
    exp(sigma g); scores are heavy-tailed, as sums of attention probabilities are."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 20230614)
    B, Hh, n, d, dt = c["batch"], c["heads"], c["n"], c["d"], DT[c["dtype"]]
    T = c["steps"] if c["kind"] == "generation" else TOKENS if c["kind"] == "step" else 1
    x = {}
    if c["kind"] not in ("step", "compress"):
        x["Q"] = _randn(gen, B, Hh, n, d).to(dt)
    x["K"] = (_randn(gen, B, Hh, n, d) * torch.exp(c["sigma"] * _randn(gen, B, Hh, n, 1))).to(dt)
    x["V"] = _randn(gen, B, Hh, n, d).to(dt)
    if c["kind"] != "compress":
        x["q"] = _randn(gen, T, B, Hh, d).to(dt)
        x["k"] = (_randn(gen, T, B, Hh, d) * torch.exp(c["sigma"] * _randn(gen, T, B, Hh, 1))).to(dt)
        x["v"] = _randn(gen, T, B, Hh, d).to(dt)
    if c["kind"] in ("step", "compress"):
        x["score"] = torch.exp(1.5 * _randn(gen, B, Hh, n)) * 0.3
    return x


def prepare(case, seed):
    c, x = case, _inputs(case, seed)
    B, Hh, n, d, dt = c["batch"], c["heads"], c["n"], c["d"], DT[c["dtype"]]
    cache = h2o.H2OCache(B, Hh, d, c["heavy"], c["recent"], dt, device=DEV, rank=c["rank"],
                         kv_bits=c["kv_bits"])
    s = dict(kind=c["kind"], cache=cache, x=x, n=n, chunk=c["chunk"], i=0)
    if c["kind"] == "step":
        # a full cache: the n = heavy + recent tokens of the prompt, with their scores
        cache.prefill_select(x["K"], x["V"], x["score"])
        del x["K"], x["V"], x["score"]
    if c["kind"] in ("step", "compress"):
        s["state"] = cache.views()
    if c["kind"] != "compress":
        T = len(x["q"])
        s["out"] = torch.empty((T, B, Hh, d), dtype=dt, device=DEV)
        s["tokens"] = [(x["q"][t], x["k"][t], x["v"][t], s["out"][t]) for t in range(T)]
    if c["kind"] in ("scores", "attention", "generation"):
        s["colsum"] = torch.empty((B, Hh, n), dtype=torch.float32, device=DEV)
    if c["kind"] == "attention":
        s["attn"] = torch.empty((B, Hh, n, d), dtype=dt, device=DEV)
        s["ws"] = torch.empty(h2o.h2o_prefill_attention_workspace_bytes(cache.cfg, n),
                              dtype=torch.uint8, device=DEV)
    if c["kind"] == "chunked":
        m = c["chunk"]
        s["pieces"] = [tuple(x[w][:, :, a:a + m].contiguous() for w in "QKV") for a in range(0, n, m)]
        s["outs"] = [torch.empty_like(p[0]) for p in s["pieces"]]
    return s


# ---- one pass ----------------------------------------------------------------------------
def run(state):
    s, cache = state, state["cache"]
    kind = s["kind"]
    if kind == "step":
        # the next token; the outputs are what the program reads, and the cache it has updated
        q, k, v, out = s["tokens"][s["i"]]
        s["i"] = (s["i"] + 1) % TOKENS
        cache.decode_step(q, k, v, out)
        return [out, *s["state"]]
    x = s["x"]
    cache.reset()
    if kind == "compress":
        cache.prefill_select(x["K"], x["V"], x["score"])
        return list(s["state"])
    if kind == "chunked":
        for (Q, K, V), out in zip(s["pieces"], s["outs"]):
            cache.prefill_chunk(Q, K, V, out=out)
        got = list(s["outs"])
    elif kind == "attention":
        h2o.h2o_prefill_attention_scores(cache.handle, x["Q"], x["K"], x["V"], s["n"], s["ws"],
                                         s["ws"].numel(), s["attn"], s["colsum"])
        got = [s["attn"], s["colsum"]]
    else:
        cache.prefill_scores(x["Q"], x["K"], x["V"], colsum_out=s["colsum"])
        got = [s["colsum"]]
    # The first generated token (generation: all of them).  What the prompt phase left in the
    # cache shows in these outputs; the slots themselves are not returned, because two tokens
    # whose scores agree to rounding may change places at the threshold, and every later slot
    # of that head would then hold its neighbour (the compress case returns them, exactly).
    for q, k, v, out in s["tokens"]:
        cache.decode_step(q, k, v, out)
    return got + [s["out"]]


# ---- what a pass cannot do without ---------------------------------------------------------
def _rows(c, count):
    """Bytes of `count` cached (key, value) row pairs per head, over all heads."""
    es = 4 if c["dtype"] == "f32" else 2
    row = c["d"] // 2 + 8 * (c["d"] // 64) if c["kv_bits"] == 4 else c["d"] * es
    return c["batch"] * c["heads"] * count * 2 * row


def _step_work(c, slots):
    es = 4 if c["dtype"] == "f32" else 2
    heads = c["batch"] * c["heads"]
    # rows, scores (read and written), positions, the token's q / k / v / out and its stored row
    by = _rows(c, slots) + heads * (12 * slots + 4 * c["d"] * es + 8) + _rows(c, 1)
    return by, heads * 4.0 * (slots + 1) * c["d"]


def work(case):
    c = case
    es = 4 if c["dtype"] == "f32" else 2
    heads, n, d = c["batch"] * c["heads"], c["n"], c["d"]
    k = c["heavy"] + c["recent"]
    if c["kind"] == "step":
        by, fl = _step_work(c, k)
        return {"bytes": by, "flops": fl}
    kept = min(n, k)
    gather = 2 * _rows(c, kept) + heads * (4 * n + 8 * kept)
    if c["kind"] == "compress":
        return {"bytes": gather, "flops": 0}
    by, fl = gather + heads * (2 * n * d * es + 4 * n), 0.0     # Q, K read, column sums written
    pairs = n * (n + 1) / 2.0
    if c["kind"] == "chunked":
        pairs, seen = 0.0, 0
        for a in range(0, n, c["chunk"]):
            m = min(c["chunk"], n - a)
            pairs += m * min(seen, k) + m * (m + 1) / 2.0
            seen += m
    fl += heads * 2.0 * pairs * d                               # Q K^T
    if c["kind"] in ("attention", "chunked"):
        fl += heads * 2.0 * pairs * d                           # P V
        by += heads * 2 * n * d * es                            # V read, attention output written
    for t in range(c["steps"]):
        b, f = _step_work(c, min(k, n + t))
        by, fl = by + b, fl + f
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # About four times what the outputs differ from float64 by (measured on each kind): outputs
    # are rounded once to their 16-bit type (f16 1.8e-4, bf16 1.3e-3 relative); binary32 outputs,
    # scores and column sums are at 1e-7 and move with the order of their sums.  "max" leaves room for one element's rounding and, behind a prompt
    # phase, for one head that keeps another of two tokens with equal scores.
    c = case
    if c["kind"] == "compress":
        return "exact"
    if c["kind"] == "step":
        if c["dtype"] == "f32":
            return {"rel": 2e-6, "max": 2e-5}
        return {"rel": 1e-3, "max": 4e-3} if c["dtype"] == "f16" else {"rel": 5e-3, "max": 3e-2}
    if c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 2e-3, "max": 0.25} if c["dtype"] == "f16" else {"rel": 6e-3, "max": 0.25}


# ---- float64 -------------------------------------------------------------------------------
def _quantised(x):
    """Rows as the 4-bit cache stores them: groups of 64, min-max, binary32 operations."""
    g = x.float().unflatten(-1, (-1, 64))
    mn, mx = g.amin(-1, keepdim=True), g.amax(-1, keepdim=True)
    sc = (mx - mn) / torch.full_like(mx, 15.0)     # (a scalar divisor would become a product)
    code = torch.where(sc > 0, ((g - mn) / sc).round().clamp(0, 15), torch.zeros_like(g))
    return (mn.double() + code.double() * sc.double()).flatten(-2)


def _ranked(c, acc, pos, t):
    return acc / (t - pos + 1).double() if c["rank"] == 1 else acc


def _exact_step(c, K, V, acc, pos, t, q, k, v):
    """One step on a full cache: [heads, slots, d] rows, [heads, slots] scores and positions
    (updated in place); returns the output [heads, d]."""
    scale = 1.0 / math.sqrt(c["d"])
    q, k, v = q.double(), k.double(), v.double()
    s = torch.matmul(K, q.unsqueeze(-1)).squeeze(-1) * scale
    p = torch.softmax(torch.cat([s, (q * k).sum(-1, keepdim=True) * scale], -1), -1)
    out = torch.matmul(p[:, None, :-1], V).squeeze(1) + p[:, -1:] * v
    acc += p[:, :-1]
    r = _ranked(c, acc, pos, t).masked_fill(pos > t - c["recent"], math.inf)
    h = torch.arange(len(q), device=q.device)
    best = r.amin(-1, keepdim=True)
    slot = torch.where(r == best, pos, torch.full_like(pos, 2 ** 31 - 1)).argmin(-1)
    new_k, new_v = (_quantised(k), _quantised(v)) if c["kv_bits"] == 4 else (k, v)
    K[h, slot], V[h, slot], acc[h, slot], pos[h, slot] = new_k, new_v, p[:, -1], t
    return out


def _exact_keep(c, score, pos, t_new):
    """Indices [heads, kept] (ascending) of what the compression keeps of candidates in position order."""
    n, k = score.shape[-1], c["heavy"] + c["recent"]
    if n <= k:
        return torch.arange(n, device=score.device).expand(len(score), n)
    r = _ranked(c, score, pos, t_new - 1)
    r = r.masked_fill(pos >= t_new - c["recent"], math.inf)
    # a stable ascending sort drops the lowest, and of equal ones the earlier positions
    order = r.sort(dim=-1, stable=True).indices[:, n - k:]
    return order.sort(dim=-1).values


def _exact_chunk(c, Q, K, V, want_out):
    """Softmax of the last len(Q) positions over K's, per head: (output, column sums)."""
    scale, m, n = 1.0 / math.sqrt(c["d"]), Q.shape[-2], K.shape[-2]
    outs, sums = [], []
    hidden = torch.ones(m, n, dtype=torch.bool, device=Q.device).triu(n - m + 1)
    for q, k, v in zip(Q, K, V):
        p = torch.matmul(q.double(), k.double().t()).mul_(scale).masked_fill_(hidden, -math.inf)
        p = torch.softmax(p, -1)
        sums.append(p.sum(0))
        if want_out:
            outs.append(torch.matmul(p, v.double()))
        del p
    return (torch.stack(outs) if want_out else None), torch.stack(sums)


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    B, Hh, n, d = c["batch"], c["heads"], c["n"], c["d"]
    heads, k = B * Hh, c["heavy"] + c["recent"]
    flat = {w: y.flatten(0, 1) if y.dim() == 4 and w in "QKV" else y for w, y in x.items()}
    token = [tuple(x[w][t].flatten(0, 1) for w in "qkv") for t in range(len(x["q"]))] if "q" in x else []
    pos = torch.arange(n, device=DEV).expand(heads, n)
    shaped = lambda y: y.unflatten(0, (B, Hh))  # noqa: E731
    if c["kind"] == "step":
        stored = (lambda y: _quantised(y)) if c["kv_bits"] == 4 else (lambda y: y.double())
        K, V = stored(flat["K"]), stored(flat["V"])
        acc, p = x["score"].flatten(0, 1).double(), pos.clone()
        out = _exact_step(c, K, V, acc, p, n, *token[0])
        rows = [None, None] if c["kv_bits"] == 4 else [shaped(K), shaped(V)]
        return [shaped(out), *rows, shaped(acc), shaped(p).int()]
    if c["kind"] == "compress":
        at = _exact_keep(c, x["score"].flatten(0, 1), pos, n)
        row = at.unsqueeze(-1).expand(-1, -1, d)
        return [shaped(flat["K"].gather(1, row)), shaped(flat["V"].gather(1, row)),
                shaped(x["score"].flatten(0, 1).gather(1, at)), shaped(at).int()]
    got = []
    if c["kind"] == "chunked":
        K = torch.empty(heads, 0, d, device=DEV, dtype=torch.float64)
        V, acc, p, t = K, K[..., 0], K[..., 0].long(), 0
        for a in range(0, n, c["chunk"]):
            b = min(n, a + c["chunk"])
            K, V = (torch.cat([y, flat[w][:, a:b].double()], 1) for y, w in ((K, "K"), (V, "V")))
            out, sums = _exact_chunk(c, flat["Q"][:, a:b], K, V, True)
            acc = sums + torch.cat([acc, torch.zeros(heads, b - a, device=DEV, dtype=torch.float64)], 1)
            p, t = torch.cat([p, pos[:, a:b]], 1), b
            at = _exact_keep(c, acc, p, t)
            row = at.unsqueeze(-1).expand(-1, -1, d)
            K, V, acc, p = K.gather(1, row), V.gather(1, row), acc.gather(1, at), p.gather(1, at)
            got.append(shaped(out))
    else:
        attn, sums = _exact_chunk(c, flat["Q"], flat["K"], flat["V"], c["kind"] == "attention")
        got = ([shaped(attn)] if attn is not None else []) + [shaped(sums)]
        at = _exact_keep(c, sums, pos, n)
        row = at.unsqueeze(-1).expand(-1, -1, d)
        K, V = flat["K"].gather(1, row).double(), flat["V"].gather(1, row).double()
        acc, p, t = sums.gather(1, at), at.clone(), n
    outs = []
    for i, (q, kn, vn) in enumerate(token):
        if K.shape[1] < k:          # a free slot: no eviction yet
            return None
        outs.append(_exact_step(c, K, V, acc, p, t + i, q, kn, vn))
    return got + [torch.stack([shaped(y) for y in outs])]
