"""What the framework is timed on: calls as a serving program makes them, over the range of sizes it meets.

A unit is one KV-head cache (one layer, one sequence, one KV head).  A model calls the path layer by
layer, so an ordinary call has batch x KV heads units: 8 for one Llama-3-8B-shaped sequence, 256 for
a batch of 32.  Whole-model calls (every layer's units at once, as replayed caches are evaluated)
have thousands.  The kinds of call:

  attend   one decode step of certified attention over retained caches (ebd_attend_certify)
  evict    the sampler: inclusion probabilities, mask, compaction (ebd_evict)
  scores   importance scores from a window of queries or the last prefill queries (ebd_scores)
  blocks   per-block variance contributions, the fine-grained probe (ebd_block_contributions)
  request  one layer's share of a request: scores, eviction, then six decode steps (append,
           certified attention, running certificate) through the allocating helpers

Buffers, parameter structs and workspaces are made in prepare(), as a serving program keeps them.
"""
import math

import torch

import paper_2607_21475_amd as ebd
from paper_2607_21475_amd import cache

D = ebd.HEAD_DIM
SINK, RECENT = 4, 64
MIXED = (0.05, 0.10, 0.15, 0.25, 0.50)  # the budgets of the replay grid
STEPS = 6  # decode steps the deployed certificate covers
BLOCK = 64  # positions per block of the fine-grained probe
SEED = 20260721  # the sampler's seed: fixed, so that the same scores keep the same rows


def _case(name, kind, units, n, group=4, budget=0.25, ragged=False, mixed=False, eps=0.01,
          heavy_tail=False, queries=32, causal=False, design=0, offset=True):
    c = dict(kind=kind, units=units, n=n, group=group, budget=budget, ragged=ragged, mixed=mixed,
             eps=eps, heavy_tail=heavy_tail, queries=queries, causal=causal, design=design,
             offset=offset)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one layer of one sequence at a short context, 8 KV heads = 8 query heads: pure latency
        _case("attend_layer_b1_4k", "attend", 8, 4096, group=1, budget=0.10),
        # one layer of one long-context sequence: few units, many rows each
        _case("attend_layer_b1_128k", "attend", 8, 131072, budget=0.10, eps=0.005, heavy_tail=True),
        # one Qwen2.5-7B-shaped layer (4 KV heads, 7 query heads each), batch 16, requests of
        # different lengths and budgets
        _case("attend_layer_b16_ragged", "attend", 64, 6144, group=7, ragged=True, mixed=True),
        # one Llama-3-8B-shaped layer, batch 32, 16384 tokens: the ordinary serving step
        _case("attend_layer_b32_16k", "attend", 256, 16384),
        # the same model's caches of all 32 layers in one call, the largest step
        _case("attend_model_b32_16k", "attend", 8192, 16384),
        # the eviction after the prefill of one short sequence, one layer
        _case("evict_layer_b1_4k", "evict", 8, 4096, budget=0.10),
        # ... of one layer of a batch of four long-context sequences
        _case("evict_layer_b4_128k", "evict", 32, 131072, budget=0.10, eps=0.005, heavy_tail=True),
        # ... of one Llama-3-8B-shaped layer, batch 32
        _case("evict_layer_b32_16k", "evict", 256, 16384),
        # a chunk of replay cells: lengths of 2k to 16k and every budget, 126 cells x 8 heads
        _case("evict_replay_ragged", "evict", 1008, 16384, ragged=True, mixed=True),
        # importance scores of one Llama-3-8B-shaped layer, batch 32, a 32-query window
        _case("scores_layer_b32_16k", "scores", 256, 16384, queries=32),
        # the fine-grained probe over one Qwen2.5-7B-shaped layer, batch 16
        _case("blocks_layer_b16_6k", "blocks", 64, 6144, group=7),
        # one layer of one sequence from scores to the certificate
        _case("request_layer_b1_8k", "request", 8, 8192, budget=0.25),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attend", "attend", "evict", "evict", "scores", "blocks", "request"])
    n = _log(rng, 512, 131072)
    limit = {"attend": 24e6, "evict": 4.5e6, "scores": 4.5e6, "blocks": 4e6, "request": 3e5}[kind]
    units = min(_log(rng, 1, 2048), max(1, int(limit / n)))
    heavy = rng.random() < 0.4
    return _case(None, kind, units, n, group=rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 12]),
                 budget=round(rng.uniform(0.05, 0.5), 3), ragged=rng.random() < 0.5,
                 mixed=rng.random() < 0.3, eps=0.005 if heavy else 0.01, heavy_tail=heavy,
                 queries=rng.choice([8, 16, 29, 32, 48, 64, 96, 128]), causal=rng.random() < 0.4,
                 design=rng.choice([0, 0, 0, 1, 2, 3]), offset=rng.random() < 0.85)


# ---- sizes -----------------------------------------------------------------------------------

def _lengths(c):
    """Unit lengths: all n, or spread over [n / 8, n] in odd steps."""
    if not c["ragged"]:
        return [c["n"]] * c["units"]
    lo = max(1, c["n"] // 8)
    return [lo + int((c["n"] - lo) * ((0.618033988749895 * (u + 1)) % 1.0)) for u in range(c["units"])]


def _budgets(c):
    return [MIXED[u % 5] if c["mixed"] else c["budget"] for u in range(c["units"])]


def _expected(c):
    """Expected retained rows per unit."""
    out = []
    for n, f in zip(_lengths(c), _budgets(c)):
        prot = min(n, SINK + RECENT)
        out.append(min(n, prot + max(f * n - prot, c["eps"] * (n - prot), 0.0)))
    return out


def work(c):
    tokens, kept = float(sum(_lengths(c))), float(sum(_expected(c)))
    U, G = c["units"], c["group"]
    attend_b = kept * (4 * D + 4) + U * G * (2 * D + 4 * D + 16)
    attend_f = kept * (6 * D * G + 2 * D)
    evict_b = tokens * (0 if c["design"] == 3 else 4) + kept * (8 * D + 8)
    scores_b = tokens * (2 * D + 4) + U * c["queries"] * 2 * D
    scores_f = tokens * c["queries"] * 2 * D
    if c["kind"] == "attend":
        return {"bytes": attend_b + (0 if c["offset"] else U * G * 4 * D), "flops": attend_f}
    if c["kind"] == "evict":
        return {"bytes": evict_b, "flops": tokens}
    if c["kind"] == "scores":
        return {"bytes": scores_b, "flops": scores_f}
    if c["kind"] == "blocks":
        return {"bytes": kept * (4 * D + 8) + U * (G * (6 * D + 4) + 4 * _nblocks(c)),
                "flops": kept * 4 * D * G}
    return {"bytes": scores_b + evict_b + STEPS * (attend_b + U * 8 * D),
            "flops": scores_f + STEPS * attend_f}


def _nblocks(c):
    return max(1, -(-c["n"] // BLOCK))


def tolerance(c):
    # Sums in 32 bits of a few hundred to a few ten thousand exact products; the variance is a
    # difference of such sums, and the range term's weights are exponentials of them.
    if c["kind"] == "evict":
        return {"rel": 1e-6, "max": 1e-4, "differ": 0.0}
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}


# ---- inputs ----------------------------------------------------------------------------------

def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFF)
    return g


def _normal(shape, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _offsets(sizes):
    off = [0]
    for s in sizes:
        off.append(off[-1] + int(s))
    return off


def _dev(values, dtype):
    return torch.tensor(values, dtype=dtype, device="cuda")


def _draw_scores(c, shape, heavy, g):
    """Importance scores: attention mass is log-normal-like; long contexts take Pareto(1.5)
    scores that are independent of the keys; heavy-hitter keys score high."""
    if c["heavy_tail"]:
        u = torch.rand(shape, generator=g, device="cuda")
        return torch.pow((1.0 - u).clamp_min(1e-7), -1.0 / 1.5)
    s = torch.exp(torch.randn(shape, generator=g, device="cuda")) * 1e-3
    return torch.where(heavy, s * 30.0, s)


def _solve(s, tail, m, eps):
    """lambda with sum over the tail of clip(lambda s, eps, 1) = m, per row of s."""
    pos = tail & (s > 0)
    npos, ntail = pos.sum(1).to(s.dtype), tail.sum(1).to(s.dtype)
    lo = torch.zeros_like(m)
    big = torch.where(pos, s, torch.full_like(s, math.inf)).min(1).values
    hi = torch.where(torch.isfinite(big), 1.0 / big.clamp_min(1e-30), torch.ones_like(big))
    for _ in range(64 if s.dtype == torch.float64 else 40):
        mid = 0.5 * (lo + hi)
        v = (s * mid[:, None]).clamp(eps, 1.0)
        less = torch.where(tail, v, torch.zeros_like(v)).sum(1) < m
        lo, hi = torch.where(less, mid, lo), torch.where(less, hi, mid)
    lam = hi
    for _ in range(3):  # the exact solve of the piece that the bisection ended on
        p = s * lam[:, None]
        H = (tail & (p >= 1)).sum(1).to(s.dtype)
        Lo = (tail & (p <= eps)).sum(1).to(s.dtype)
        S = torch.where(tail & (p < 1) & (p > eps), s, torch.zeros_like(s)).sum(1)
        lam = torch.where(S > 0, (m - H - eps * Lo) / S.clamp_min(1e-300 if s.dtype == torch.float64 else 1e-37), lam)
    lam = torch.where(m <= eps * ntail, torch.zeros_like(lam), lam)
    return torch.where((m > eps * ntail) & (m >= npos + eps * (ntail - npos)),
                       torch.full_like(lam, math.inf), lam)


def _inclusion(s, tail, lam, eps):
    p = torch.where(s > 0, s * lam[:, None], torch.zeros_like(s)).clamp(eps, 1.0)
    return torch.where(tail, p, torch.ones_like(p))


def _masks(lengths, width):
    n = _dev(lengths, torch.int64)[:, None]
    i = torch.arange(width, device="cuda")[None, :]
    real = i < n
    return real, real & (i >= SINK) & (i < n - RECENT)


def _chunks(lengths):
    """Runs of units whose padded size stays moderate."""
    u = 0
    while u < len(lengths):
        v, w = u + 1, lengths[u]
        while v < len(lengths) and max(w, lengths[v]) * (v + 1 - u) <= 1 << 25:
            w = max(w, lengths[v])
            v += 1
        yield u, v, w
        u = v


def _keys(rows, heavy, g):
    k = _normal((rows, D), g)
    return k.mul_(torch.where(heavy, 4.0, 1.0).to(torch.bfloat16)[:, None])


def _retained(c, seed):
    """Retained caches as an eviction leaves them: rows, their probabilities and positions."""
    lengths, budgets = _lengths(c), _budgets(c)
    cap = cache.plan_capacity(lengths, budgets, SINK, RECENT, pi_min=c["eps"])
    rows, U = cap[-1], c["units"]
    g = _gen(seed, 1)
    pic = torch.zeros(rows, device="cuda")
    idx = torch.zeros(rows, dtype=torch.int32, device="cuda")
    heavy = torch.zeros(rows, dtype=torch.bool, device="cuda")
    count = torch.zeros(U, dtype=torch.int32, device="cuda")
    cap_off = _dev(cap, torch.int64)
    for a, b, w in _chunks(lengths):
        real, tail = _masks(lengths[a:b], w)
        hh = torch.rand((b - a, w), generator=g, device="cuda") < 0.02
        s = _draw_scores(c, (b - a, w), hh, g)
        n = _dev(lengths[a:b], torch.float32)
        m = _dev(budgets[a:b], torch.float32) * n - torch.minimum(n, torch.full_like(n, SINK + RECENT))
        p = _inclusion(s, tail, _solve(s, tail, m, c["eps"]), c["eps"])
        keep = real & (torch.rand(p.shape, generator=g, device="cuda") < p)
        rank = keep.cumsum(1) - 1
        keep &= rank < (cap_off[a + 1:b + 1] - cap_off[a:b])[:, None]
        at = (cap_off[a:b, None] + rank)[keep]
        pic[at] = p[keep]
        heavy[at] = hh[keep]
        idx[at] = torch.arange(w, dtype=torch.int32, device="cuda").expand(b - a, w)[keep]
        count[a:b] = keep.sum(1).to(torch.int32)
    return dict(K=_keys(rows, heavy, g), V=_normal((rows, D), g), pi=pic, idx=idx, count=count,
                cap_off=cap_off, max_cap=max(y - x for x, y in zip(cap[:-1], cap[1:])),
                q=_normal((U, c["group"], D), g))


def _attend_out(c):
    U, G = c["units"], c["group"]
    f = dict(device="cuda", dtype=torch.float32)
    return dict(y=torch.zeros((U, G, D), **f), vhat=torch.zeros((U, G), **f),
                lse=torch.zeros((U, G), **f), b=torch.zeros((U, G), **f), r=torch.zeros((U, G), **f),
                status=torch.zeros(U, dtype=torch.int32, device="cuda"))


def _full(c, seed, extra=0):
    """Full caches with scores, and room for what an eviction retains of them."""
    lengths, budgets, U = _lengths(c), _budgets(c), c["units"]
    off = _offsets(lengths)
    g = _gen(seed, 2)
    heavy = torch.rand(off[-1], generator=g, device="cuda") < 0.02
    cap = cache.plan_capacity(lengths, budgets, SINK, RECENT, extra, c["eps"])
    rows = cap[-1]
    z = dict(device="cuda")
    s = dict(K=_keys(off[-1], heavy, g), V=_normal((off[-1], D), g),
             scores=_draw_scores(c, (off[-1],), heavy, g), seq_off=_dev(off, torch.int64),
             cap_off=_dev(cap, torch.int64), max_cap=max(y - x for x, y in zip(cap[:-1], cap[1:])),
             budgets=_dev(budgets, torch.float32) if c["mixed"] else None)
    s["rc"] = cache.RetainedCache(
        Kc=torch.zeros((rows, D), dtype=torch.bfloat16, **z),
        Vc=torch.zeros((rows, D), dtype=torch.bfloat16, **z), pic=torch.zeros(rows, **z),
        idxc=torch.zeros(rows, dtype=torch.int32, **z), count=torch.zeros(U, dtype=torch.int32, **z),
        status=torch.zeros(U, dtype=torch.int32, **z), cap_off=s["cap_off"], max_cap=s["max_cap"],
        lam=torch.zeros(U, **z))
    s["p"] = ebd.evict_params(U, max(lengths), s["max_cap"], s["seq_off"], s["cap_off"], SINK, RECENT,
                              c["budget"], s["budgets"], c["eps"], 0, SEED, None, 0, c["design"])
    s["ws"] = ebd.workspace(ebd.ebd_workspace_size(ebd.EBD_WS_EVICT, s["p"]))
    return s


def _query_calls(c, g):
    """Query windows of at most 64 queries per call, and the last row each query sees."""
    lengths, calls, done = _lengths(c), [], 0
    while done < c["queries"]:
        w = min(64, c["queries"] - done)
        pos = None
        if c["causal"]:  # the last prefill queries, each at its own position
            pos = _dev([[max(n - c["queries"] + done + i, 0) for i in range(w)] for n in lengths],
                       torch.int32)
        calls.append((_normal((c["units"], w, D), g), pos))
        done += w
    return calls


def prepare(c, seed):
    kind, U, G = c["kind"], c["units"], c["group"]
    if kind == "attend":
        s = _retained(c, seed)
        s["out"] = _attend_out(c)
        s["p"] = ebd.attend_params(U, G, s["max_cap"], s["cap_off"],
                                   flags=0 if c["offset"] else ebd.EBD_F_NO_OFFSET)
        s["ws"] = ebd.workspace(ebd.ebd_workspace_size(ebd.EBD_WS_ATTEND, s["p"]))
    elif kind == "evict":
        s = _full(c, seed)
    elif kind == "scores":
        lengths = _lengths(c)
        off = _offsets(lengths)
        g = _gen(seed, 3)
        heavy = torch.rand(off[-1], generator=g, device="cuda") < 0.02
        s = dict(K=_keys(off[-1], heavy, g), seq_off=_dev(off, torch.int64),
                 scores=torch.zeros(off[-1], device="cuda"), calls=[])
        for i, (q, pos) in enumerate(_query_calls(c, g)):
            p = ebd.scores_params(U, q.shape[1], max(lengths), s["seq_off"], pos, accumulate=i > 0)
            s["calls"].append((p, q, pos, ebd.workspace(ebd.ebd_workspace_size(ebd.EBD_WS_SCORES, p))))
    elif kind == "blocks":
        s = _retained(c, seed)
        o = _attend_out(c)
        p = ebd.attend_params(U, G, s["max_cap"], s["cap_off"])
        ws = ebd.workspace(ebd.ebd_workspace_size(ebd.EBD_WS_ATTEND, p))
        ebd.ebd_attend_certify(p, s["q"], s["K"], s["V"], s["pi"], s["count"], o["y"], o["vhat"],
                               o["lse"], ws)
        # the probe's inputs at the attention's own precision, but not its last bits, so that the
        # probe alone is what the outputs show
        s["y"] = (o["y"] * 4096).round() / 4096
        s["lse"] = (o["lse"] * 4096).round() / 4096
        s["blocks"] = torch.zeros((U, _nblocks(c)), device="cuda")
    else:
        s = _full(c, seed, extra=STEPS)
        g = _gen(seed, 4)
        s["calls"] = _query_calls(c, g)
        s["k_new"], s["v_new"] = _normal((STEPS, U, D), g), _normal((STEPS, U, D), g)
        s["q"] = [_normal((U, G, D), g) for _ in range(STEPS)]
        s["pos"] = [_dev([n + t for n in _lengths(c)], torch.int32) for t in range(STEPS)]
        s["unit_seq"] = _dev([u // 8 for u in range(U)], torch.int32)
        s["head0"] = _dev([(u % 8) * G for u in range(U)], torch.int32)
        s["cert"] = torch.zeros((U + 7) // 8, device="cuda")
        s["sws"] = s["aws"] = None
    s["case"] = c
    return s


# ---- one pass --------------------------------------------------------------------------------

def _evict(s):
    rc = s["rc"]
    ebd.ebd_evict(s["p"], s["scores"], s["K"], s["V"], rc.Kc, rc.Vc, rc.pic, rc.idxc, rc.count,
                  rc.status, s["ws"], lambda_out=rc.lam)
    return dict(Kc=rc.Kc, Vc=rc.Vc, pic=rc.pic, idxc=rc.idxc, count=rc.count, status=rc.status,
                lam=rc.lam)


def run(s):
    c = s["case"]
    kind, U, G = c["kind"], c["units"], c["group"]
    if kind == "attend":
        o = s["out"]
        ebd.ebd_attend_certify(s["p"], s["q"], s["K"], s["V"], s["pi"], s["count"], o["y"], o["vhat"],
                               o["lse"], s["ws"], brange=o["b"], radius=o["r"], status=o["status"])
        return o
    if kind == "evict":
        return _evict(s)
    if kind == "scores":
        for p, q, _, ws in s["calls"]:
            ebd.ebd_scores(p, q, s["K"], s["scores"], ws)
        return {"scores": s["scores"]}
    if kind == "blocks":
        ebd.ebd_block_contributions(U, G, _nblocks(c), s["max_cap"], s["cap_off"], s["q"], s["K"],
                                    s["V"], s["pi"], s["idx"], s["count"], s["y"], s["lse"],
                                    s["blocks"], block_rows=BLOCK)
        return {"blocks": s["blocks"]}
    longest = s["p"].max_rows
    for i, (q, pos) in enumerate(s["calls"]):
        _, s["sws"] = cache.importance_scores(s["K"], s["seq_off"], q, longest, pos, s["scores"],
                                              accumulate=i > 0, ws=s["sws"])
    out = _evict(s)
    s["cert"].zero_()
    steps, rc = [], s["rc"]
    for t in range(STEPS):
        ebd.ebd_append_certain(U, s["cap_off"], rc.count, s["k_new"][t], s["v_new"][t], rc.Kc, rc.Vc,
                               rc.pic, rc.idxc, s["pos"][t], rc.status)
        o = cache.attend_certify(rc, s["q"][t], ws=s["aws"])
        s["aws"] = o.pop("ws")
        ebd.ebd_certificate_step(U, G, s["cert"].shape[0], s["unit_seq"], o["r"], s["cert"],
                                 unit_head0=s["head0"])
        steps.append(o)
    return dict(out, scores=s["scores"], steps=steps, cert=s["cert"])


# ---- the same in 64 bits ---------------------------------------------------------------------

def _exact_attend(q, K, V, pi, offset=True):
    """y, Vhat, ln N, b, r of one unit (eq. (3), Theorem 2, eq. (4) at delta = 0.1)."""
    q, K, V, pi = q.double(), K.double(), V.double(), pi.double()
    logit = q @ K.T.contiguous() / math.sqrt(D)
    lw = logit - torch.log(pi)[None, :]
    lse = torch.logsumexp(lw, 1)
    w = torch.exp(lw - lse[:, None])
    y = w @ V
    d2 = (V.square().sum(1)[None, :] - 2.0 * (y @ V.T.contiguous()) + y.square().sum(1)[:, None]).clamp_min(0.0)
    kap = (1.0 - pi)[None, :] * w.square() * d2
    vhat = kap.sum(1)
    b = kap.max(1).values.sqrt()
    ld = math.log(1.0 / 0.1)
    r = (torch.sqrt(2.0 * vhat * ld) + b * ld) / (y.square().sum(1).sqrt() + 1e-9)
    if not offset:
        lse = torch.logsumexp(logit, 1)
        y = torch.exp(logit - lse[:, None]) @ V
    return y, vhat, lse, b, r, kap


def _exact_steps(q, K, V, pi, count, cap_off, offset=True):
    res, cnt, off = [], count.tolist(), cap_off.tolist()
    for u, n in enumerate(cnt):
        sl = slice(off[u], off[u] + n)
        res.append(_exact_attend(q[u], K[sl], V[sl], pi[sl], offset)[:5])
    return {k: torch.stack([x[i] for x in res]) for i, k in enumerate(("y", "vhat", "lse", "b", "r"))}


def _philox(units, groups):
    """The four Philox4x32-10 words of (token group, unit) at epoch 0, as int64 tensors."""
    mask = 0xFFFFFFFF
    c0 = torch.arange(groups, device="cuda")[None, :].expand(len(units), groups)
    c1 = _dev(units, torch.int64)[:, None].expand_as(c0)
    c2, c3 = torch.zeros_like(c0), torch.full_like(c0, 0x45424431)
    k0, k1 = SEED & mask, SEED >> 32

    def mul(a, x):  # high and low word of a 32 x 32 product, in 16-bit halves
        lo, hi = (a & 0xFFFF) * x, (a >> 16) * x
        low = lo + ((hi & 0xFFFF) << 16)
        return ((hi >> 16) + (low >> 32)) & mask, low & mask

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c0)
        h1, l1 = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return torch.stack([c0, c1, c2, c3], 2).reshape(len(units), -1)


def _exact_evict(c, s):
    """The sampler in 64 bits: lambda, and the probabilities of the rows it keeps, in their slots."""
    lengths, budgets, U = _lengths(c), _budgets(c), c["units"]
    off = _offsets(lengths)
    lam_out = torch.zeros(U, dtype=torch.float64, device="cuda")
    pic = torch.zeros(s["rc"].pic.shape[0], dtype=torch.float64, device="cuda")
    idx = torch.zeros(s["rc"].pic.shape[0], dtype=torch.int64, device="cuda")
    count = torch.zeros(U, dtype=torch.int64, device="cuda")
    for a, b, w in _chunks([4 * n for n in lengths]):
        w = (w // 4 + 3) // 4 * 4
        real, tail = _masks(lengths[a:b], w)
        sc = torch.zeros((b - a, w), dtype=torch.float64, device="cuda")
        sc[real] = s["scores"][off[a]:off[b]].double()
        if c["design"] == 3:
            sc = torch.ones_like(sc)
        n = _dev(lengths[a:b], torch.float64)
        f = _dev(budgets[a:b], torch.float32).double()
        m = f * n - torch.minimum(n, torch.full_like(n, SINK + RECENT))
        eps = float(torch.tensor(c["eps"], dtype=torch.float32))
        lam = _solve(sc, tail, m, eps)
        lam_out[a:b] = lam
        p = _inclusion(sc, tail, lam, eps)
        p32 = _inclusion(sc.float(), tail, lam.float(), eps)
        keep = real & (_philox(list(range(a, b)), w // 4).double() < p32.double() * 4294967296.0)
        at = (s["cap_off"][a:b, None] + keep.cumsum(1) - 1)[keep]
        pic[at] = p[keep]
        idx[at] = torch.arange(w, device="cuda").expand(b - a, w)[keep]
        count[a:b] = keep.sum(1)
    return lam_out, pic, idx, count


def _exact_scores(c, s):
    off, out = _offsets(_lengths(c)), []
    calls = [(x[1], x[2]) if len(x) == 4 else x for x in s["calls"]]
    for u in range(c["units"]):
        k = s["K"][off[u]:off[u + 1]].double()
        tot = torch.zeros(k.shape[0], dtype=torch.float64, device="cuda")
        for q, pos in calls:
            lg = q[u].double() @ k.T.contiguous() / math.sqrt(D)
            if pos is not None:
                lg = lg.masked_fill(torch.arange(k.shape[0], device="cuda")[None, :] > pos[u].long()[:, None],
                                    -math.inf)
            tot += torch.softmax(lg, 1).sum(0)
        out.append(tot)
    return torch.cat(out)


def exact(c, seed):
    s = prepare(c, seed)
    if c["kind"] == "attend":
        e = _exact_steps(s["q"], s["K"], s["V"], s["pi"], s["count"], s["cap_off"], c["offset"])
        return dict(e, status=None)
    if c["kind"] == "evict":
        if c["design"] in (1, 2):  # a fixed-size sweep and a ranking: no sums in their rows
            return None
        lam, pic, _, _ = _exact_evict(c, s)
        return dict(Kc=None, Vc=None, pic=pic, idxc=None, count=None, status=None, lam=lam)
    if c["kind"] == "scores":
        return {"scores": _exact_scores(c, s)}
    if c["kind"] == "blocks":
        out = torch.zeros(s["blocks"].shape, dtype=torch.float64, device="cuda")
        cnt, off = s["count"].tolist(), s["cap_off"].tolist()
        for u, n in enumerate(cnt):
            sl = slice(off[u], off[u] + n)
            q, K, V, pi = s["q"][u].double(), s["K"][sl].double(), s["V"][sl].double(), s["pi"][sl].double()
            y, lse = s["y"][u].double(), s["lse"][u].double()
            w = torch.exp(q @ K.T.contiguous() / math.sqrt(D) - torch.log(pi)[None, :] - lse[:, None])
            d2 = (V.square().sum(1)[None, :] - 2.0 * (y @ V.T.contiguous()) + y.square().sum(1)[:, None])
            kap = ((1.0 - pi)[None, :] * w.square() * d2.clamp_min(0.0)).sum(0)
            out[u].index_add_(0, s["idx"][sl].long() // BLOCK, kap)
        return {"blocks": out}
    if c["design"] in (1, 2):
        return None
    # a request: each stage on the exact values of the one before
    sc = _exact_scores(c, s)
    s["scores"] = sc.float()
    lam, pic, idx, count = _exact_evict(c, s)
    soff, rc, G = s["seq_off"].tolist(), s["rc"], c["group"]
    offs, cnt = s["cap_off"].tolist(), count.tolist()
    Kc, Vc = torch.zeros_like(rc.Kc), torch.zeros_like(rc.Vc)
    for u, n in enumerate(cnt):
        src = soff[u] + idx[offs[u]:offs[u] + n]
        Kc[offs[u]:offs[u] + n], Vc[offs[u]:offs[u] + n] = s["K"][src], s["V"][src]
    steps, cert = [], torch.zeros(s["cert"].shape[0], dtype=torch.float64, device="cuda")
    for t in range(STEPS):
        for u in range(c["units"]):
            at = offs[u] + cnt[u]
            Kc[at], Vc[at], pic[at] = s["k_new"][t, u], s["v_new"][t, u], 1.0
            cnt[u] += 1
        e = _exact_steps(s["q"][t], Kc, Vc, pic, _dev(cnt, torch.int64), s["cap_off"])
        head = s["head0"].long()[:, None] + torch.arange(G, device="cuda")[None, :]
        for q in range(cert.shape[0]):
            use = (s["unit_seq"] == q)[:, None] & (head % 4 == 0)
            if bool(use.any()):
                cert[q] = max(cert[q], e["r"][use].mean())
        steps.append(dict(e, status=None))
    return dict(Kc=None, Vc=None, pic=pic, idxc=None, count=None, status=None, lam=lam, scores=sc,
                steps=steps, cert=cert)
