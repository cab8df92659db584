"""Performance cases of the eviction library: what a serving program has it do,
through the binding's public calls (jacap.prepare / run_evict / run_evict_slots
/ prepare_greedy / run_greedy), over the range of sizes and options that the
workloads of this repository cover.

A case names the cache (layers, KV heads, head_dim, sequence lengths, dtype),
the observation window, the budget and the method's options. Inputs follow the
synthetic workloads' recipe: query centres, outlier channels, an attention sink
at token 0, planted heavy hitters and, for the longest contexts, a drifting key
mean; everything is drawn on the GPU from the seed.
"""

import math

import torch

from paper_2609_08131_amd import jacap

# Fields of a case and what they are when a case does not name them.
DEFAULTS = {
    "call": "evict",        # evict | slots (evicted positions, refilled in place) | greedy
    "layers": 1, "kv_heads": 8, "group": 4, "head_dim": 128, "dtype": "bf16",
    "lens": "",             # sequence lengths, comma separated, or
    "seqs": 1, "lo": 0, "hi": 0,   # that many lengths drawn from lo..hi by the case's lens_seed
    "lens_seed": 0,
    "window": 32, "budget": 512,
    "tau": 10.0, "ridge": 1.0,
    "cov": "diag",          # diag | full
    "gqa": "pooled",        # pooled | per_head
    "protect": 0,
    "drift": False,         # drifting key mean (long contexts)
    "token_major": False,   # K and V stored [L][T][H][d] and passed as views
}


def listed():
    return [
        # One short prompt of a small fp32 model: a call that is all latency.
        {"name": "short_fp32", "kv_heads": 1, "group": 1, "head_dim": 64, "dtype": "fp32",
         "lens": "512", "window": 16, "budget": 64},
        # One layer of an 8B model after an 8K prefill (evicting layer by layer).
        {"name": "layer_8k", "lens": "8192", "window": 32, "budget": 512},
        # A batch of prompts of very unequal, odd lengths (one empty, one of a
        # single token) in an fp32 cache.
        {"name": "ragged_odd_fp32", "lens": "0,1,17,255,256,257,1000,8193", "dtype": "fp32",
         "group": 2, "window": 16, "budget": 256, "protect": 64},
        # A whole 8B model after a 32K prefill.
        {"name": "model_32k", "layers": 32, "lens": "32768", "window": 32, "budget": 512},
        # The same cache with every query head of a group scored alone.
        {"name": "model_32k_per_head", "layers": 32, "lens": "32768", "window": 32, "budget": 512,
         "gqa": "per_head"},
        # A whole 8B model at 128K: the largest single context.
        {"name": "model_128k", "layers": 32, "lens": "131072", "window": 64, "budget": 1024,
         "drift": True},
        # ... with the full query covariance (Algorithm 1's literal input).
        {"name": "model_128k_full_cov", "layers": 32, "lens": "131072", "window": 64,
         "budget": 1024, "drift": True, "cov": "full"},
        # A batch of 16 ragged prompts (continuous batching).
        {"name": "ragged_16", "layers": 32, "seqs": 16, "lo": 4096, "hi": 32768, "lens_seed": 4,
         "window": 32, "budget": 256},
        # A decoding round of 16 sequences at a reserved budget of 2048: 128
        # tokens are evicted and their slots refilled in place.
        {"name": "decode_2k_slots", "call": "slots", "layers": 32,
         "lens": ",".join(["2176"] * 16), "window": 64, "budget": 2048},
        # A decoding round at a reserved budget of 16384 with a compacted cache
        # (8 layers, as one of four pipeline stages holds).
        {"name": "decode_16k_compact", "layers": 8, "lens": ",".join(["16512"] * 16),
         "window": 64, "budget": 16384},
        # Plain statistical leverage (ridge 0) of an 8K prefill: the units whose
        # capacity matrix needs the fp64 path.
        {"name": "model_8k_ridge0", "layers": 32, "lens": "8192", "window": 32, "budget": 512,
         "ridge": 0.0},
        # The exact greedy selection for one layer of an 8K prefill.
        {"name": "greedy_layer_8k", "call": "greedy", "lens": "8192", "window": 32, "budget": 512},
    ]


# The largest listed case holds this many token entries (tokens x layers x KV heads).
MOST_ENTRIES = 60_000_000


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["short", "layer", "model", "batch", "decode", "fp64", "greedy"])
    c = {"head_dim": rng.choice([64, 128, 128]), "group": rng.choice([1, 2, 4, 8]),
         "kv_heads": rng.choice([1, 2, 4, 8]), "window": rng.choice([16, 32, 64, rng.randint(5, 64)]),
         "tau": rng.choice([5.0, 10.0, 10.0, 20.0]), "ridge": rng.choice([1.0, 1.0, 0.0078125])}
    if kind == "short":
        c.update(dtype=rng.choice(["fp32", "bf16"]), lens=str(_log_int(rng, 200, 4096)),
                 budget=_log_int(rng, 16, 256), cov=rng.choice(["diag", "full"]))
    elif kind == "layer":
        n = _log_int(rng, 2048, 131072)
        c.update(lens=str(n), budget=_log_int(rng, 64, 2048), layers=rng.choice([1, 1, 2, 4]),
                 cov=rng.choice(["diag", "diag", "full"]), drift=n > 65536,
                 token_major=rng.random() < 0.5)
    elif kind == "model":
        n = _log_int(rng, 4096, 131072)
        c.update(lens=str(n), layers=rng.randint(8, 32), budget=_log_int(rng, 128, 2048),
                 gqa=rng.choice(["pooled", "pooled", "per_head"]), drift=n > 65536,
                 cov=rng.choice(["diag", "diag", "full"]))
        if c["gqa"] == "per_head":   # every query head is a unit: no more of them than listed
            c["group"] = rng.choice([2, 4])
            c["layers"] = max(1, min(c["layers"], 8_000_000 // (n * c["kv_heads"])))
    elif kind == "batch":
        c.update(seqs=rng.randint(2, 24), lo=_log_int(rng, 16, 4096), hi=_log_int(rng, 5000, 32768),
                 lens_seed=rng.randrange(1 << 20), layers=rng.randint(1, 16),
                 budget=_log_int(rng, 64, 1024), protect=rng.choice([0, 0, 16, 64]),
                 token_major=rng.random() < 0.5)
    elif kind == "decode":
        r = _log_int(rng, 1024, 16384)
        c.update(call=rng.choice(["evict", "slots"]), seqs=rng.randint(1, 16), lo=r + 128, hi=r + 128,
                 layers=rng.randint(1, 16), budget=r, protect=rng.choice([0, 64]))
    elif kind == "fp64":
        dtype = rng.choice(["fp32", "bf16"])
        c.update(dtype=dtype, lens=str(_log_int(rng, 1024, 16384)), layers=rng.randint(1, 8),
                 budget=_log_int(rng, 64, 1024))
        if dtype == "bf16":
            c["ridge"] = 0.0
    else:
        c.update(call="greedy", lens=str(_log_int(rng, 1000, 16384)), budget=_log_int(rng, 64, 512),
                 layers=rng.randint(1, 8), ridge=1.0)
    lens = _lens(_full(c))
    limit = 8_000_000 if c.get("dtype") == "fp32" else MOST_ENTRIES // 2
    c["layers"] = max(1, min(c.get("layers", 1), limit // (sum(lens) * c["kv_heads"])))
    return c


def _full(case):
    c = dict(DEFAULTS)
    c.update({k: v for k, v in case.items() if k != "name"})
    return c


def _lens(c):
    if c["lens"]:
        return [int(x) for x in c["lens"].split(",")]
    gen = torch.Generator().manual_seed(int(c["lens_seed"]))
    return [int(x) for x in torch.randint(c["lo"], c["hi"] + 1, (c["seqs"],), generator=gen)]


def _inputs(c, lens, seed):
    """Window queries [B][L][H_q][w][d], keys and values [L][H][T][d] (the
    synthetic workloads' recipe, drawn on the GPU)."""
    dev = "cuda"
    L, H, G, d, w = c["layers"], c["kv_heads"], c["group"], c["head_dim"], c["window"]
    T = sum(lens)
    dt = torch.float32 if c["dtype"] == "fp32" else torch.bfloat16
    gen = torch.Generator(device=dev).manual_seed(int(seed) & ((1 << 62) - 1))
    shape = (L, T, H, d) if c["token_major"] else (L, H, T, d)
    k_all, v_all = torch.empty(shape, dtype=dt, device=dev), torch.empty(shape, dtype=dt, device=dev)
    if c["token_major"]:
        k_all, v_all = k_all.transpose(1, 2), v_all.transpose(1, 2)
    q_all = torch.empty((len(lens), L, H * G, w, d), dtype=dt, device=dev)

    def rows(x, index):   # x [l][H][n][d], index [l][H][m] -> index for scatter / gather
        return index.unsqueeze(-1).expand(*index.shape, x.shape[-1])

    off = 0
    for b, n in enumerate(lens):
        step = max(1, min(L, (1 << 27) // max(1, H * n * d)))   # layers drawn at once
        for l0 in range(0, L, step):
            l1 = min(L, l0 + step)
            m = l1 - l0
            centre = torch.randn((m, H, d), generator=gen, device=dev)
            q = torch.randn((m, H, G, w, d), generator=gen, device=dev) + centre[:, :, None, None]
            q_all[b, l0:l1] = q.reshape(m, H * G, w, d).to(dt)
            if n == 0:
                continue
            k = torch.randn((m, H, n, d), generator=gen, device=dev)
            v = torch.randn((m, H, n, d), generator=gen, device=dev)
            kscale = torch.rand((m, 1, 1), generator=gen, device=dev) * 8.0 + 2.0
            for x, scale in ((k, kscale), (v, torch.full_like(kscale, 8.0))):
                ch = torch.rand((m, H, d), generator=gen, device=dev).argsort(-1)[..., :4]
                x *= torch.ones((m, H, d), device=dev).scatter_(2, ch, scale.expand(m, H, 4))[:, :, None]
            if c["drift"]:
                seg = torch.arange(n, device=dev) // 4096
                steps = 0.5 * torch.randn((m, H, (n + 4095) // 4096, d), generator=gen, device=dev)
                steps[:, :, 0] = 0.0
                k += torch.cumsum(steps, 2)[:, :, seg]
            heavy = min(32 if n > 1024 else 8, n - 1)
            if heavy > 0:   # distinct positions in 1 .. n-1
                part = (n - 1) / heavy
                at = torch.rand((m, H, heavy), generator=gen, device=dev) * 0.99 + torch.arange(heavy, device=dev)
                pos = 1 + (at * part).long().clamp_(0, n - 2)
                hit = centre[:, :, None] + 0.1 * torch.randn((m, H, heavy, d), generator=gen, device=dev)
                k.scatter_(2, rows(k, pos), hit)
            k[:, :, 0] = 4.0 * centre
            k_all[l0:l1, :, off:off + n] = k.to(dt)
            v_all[l0:l1, :, off:off + n] = v.to(dt)
        off += n
    return q_all, k_all, v_all


class _State:
    pass


def prepare(case, seed):
    c = _full(case)
    lens = _lens(c)
    s = _State()
    s.case = c
    s.q, s.k, s.v = _inputs(c, lens, seed)
    offs = [0]
    for n in lens:
        offs.append(offs[-1] + n)
    s.offsets = torch.tensor(offs, dtype=torch.int32, device="cuda")
    params = jacap.Params(
        budget_k=c["budget"], temperature=c["tau"], ridge=c["ridge"],
        cov_mode=jacap.COV_FULL if c["cov"] == "full" else jacap.COV_DIAG,
        gqa_mode=jacap.GQA_PER_HEAD if c["gqa"] == "per_head" else jacap.GQA_POOLED,
        protect_last=c["protect"])
    if c["call"] == "greedy":
        s.prob = jacap.prepare_greedy(s.q, s.k, s.v, s.offsets, lens, params)
    else:
        s.prob = jacap.prepare(s.q, s.k, s.v, s.offsets, lens, params)
        # rows past a sequence's length stay what the caller had there
        s.prob.k_out.zero_()
        s.prob.v_out.zero_()
        if c["call"] == "slots":
            s.slots = jacap.alloc_slots(s.prob, lens)
    return s


def run(s):
    p = s.prob
    if s.case["call"] == "greedy":
        jacap.run_greedy(p, s.q, s.k, s.v)
        return {"idx": p.idx, "order": p.order, "logdet": p.logdet}
    if s.case["call"] == "slots":
        jacap.run_evict_slots(p, s.slots, s.q, s.k, s.v)
        return {"scores": p.scores, "slots": s.slots}
    jacap.run_evict(p, s.q, s.k, s.v)
    # The retained cache holds exact copies of K and V rows: compared as the
    # stored words, not as computed numbers.
    word = torch.int32 if s.case["dtype"] == "fp32" else torch.int16
    return {"scores": p.scores, "idx": p.idx, "k": p.k_out.view(word), "v": p.v_out.view(word)}


def work(case):
    c = _full(case)
    lens = _lens(c)
    d, size = c["head_dim"], 4 if c["dtype"] == "fp32" else 2
    lh = c["layers"] * c["kv_heads"]
    entries = sum(lens) * lh
    units = len(lens) * lh
    kept = sum(min(c["budget"], n) for n in lens) * lh
    heads = c["group"] if c["gqa"] == "per_head" else 1
    # K and V once, the window queries, the index lists
    nbytes = 2 * entries * d * size + units * c["group"] * c["window"] * d * size
    kappa = 2 * d * d if c["cov"] == "full" else 3 * d
    flops = entries * heads * (2 * d + kappa)
    if c["call"] == "greedy":
        nbytes += units * c["budget"] * 8 + units * 8
        flops += entries * 2 * d + kept * 4 * d * d
        return {"bytes": nbytes, "flops": flops}
    # the symmetric Gram (half of 2 d^2) and the triangular product per token;
    # the factor and its inverse per unit
    flops += entries * heads * 2 * d * d + units * heads * 2 * d ** 3 // 3
    nbytes += entries * 4
    if c["call"] == "slots":
        nbytes += 4 * units * max(0, max(lens) - c["budget"])
    else:
        nbytes += 4 * units * c["budget"] + 2 * kept * d * size   # idx; K' and V' written
    return {"bytes": nbytes, "flops": flops}


# Scores measured against exact() over listed and drawn cases: up to 6.5e-6 in
# the 2-norm and 6e-5 in a single score (bf16 inputs; fp32 inputs 8e-8 and
# 1e-6); four times that. Positions: two scores at the edge of the budget that
# lie closer than their error may change places, which shifts the ascending
# lists (and the rows copied by them) between the two positions.
TOLERANCE = {"rel": 2.6e-5, "max": 2.5e-4, "differ": 0.01}


def tolerance(case):
    return dict(TOLERANCE)


# ---------------------------------------------------------------------------
# The method in float64 (Algorithm 1 and Eqs. 8-10), plain torch
# ---------------------------------------------------------------------------
def _weights64(c, q, k):
    """Eq. 8 weights [m][n] of m units: q [m][N][d] and k [m][n][d] in float64."""
    d, n = k.shape[-1], k.shape[1]
    mu = q.mean(1)
    x = q - mu[:, None]
    z = torch.bmm(k, mu[:, :, None].contiguous())[..., 0] / (c["tau"] * math.sqrt(d))
    if c["cov"] == "full":
        lam = torch.bmm(x.transpose(1, 2).contiguous(), x) / q.shape[1]
        kappa = (torch.bmm(k, lam) * k).sum(-1)
    else:
        kappa = torch.bmm(k * k, (x * x).mean(1)[:, :, None].contiguous())[..., 0]
    z = z - z.amax(1, keepdim=True)
    e = z.exp()
    total = e.sum(1, keepdim=True)
    top = z.argmax(1, keepdim=True)
    rest = e.scatter(1, top, 0.0).sum(1, keepdim=True)
    # 1 - alpha of the largest term is the rest of the sum over the whole
    other = (total - e).scatter(1, top, rest)
    return (e / total * (other / total)) ** 2 * kappa / d


def _scores64(c, q, k, v):
    m, n, d = v.shape
    w = _weights64(c, q, k)
    if n == 1:
        return torch.zeros_like(w)
    a = torch.bmm((v * w[..., None]).transpose(1, 2).contiguous(), v)
    a += c["ridge"] * torch.eye(d, dtype=torch.float64, device=v.device)
    low = torch.linalg.cholesky(a)
    eye = torch.eye(d, dtype=torch.float64, device=v.device).expand(m, d, d)
    inv_t = torch.linalg.solve_triangular(low, eye, upper=False).transpose(1, 2).contiguous()
    return w * torch.bmm(v, inv_t).square().sum(-1)


def _greedy64(c, q, k, v):
    """log det of the greedily chosen sets of m units."""
    m, n, d = v.shape
    w = _weights64(c, q, k)
    kk = min(c["budget"], n)
    tail = min(c["protect"], kk)
    inv = (torch.eye(d, dtype=torch.float64, device=v.device) / c["ridge"]).repeat(m, 1, 1)
    gain = (v * v).sum(-1) / c["ridge"]
    open_ = torch.ones_like(w, dtype=torch.bool)
    open_[:, n - tail:] = False
    logdet = torch.full((m,), d * math.log(c["ridge"]), dtype=torch.float64, device=v.device)
    at = torch.arange(m, device=v.device)
    for t in range(kk):
        if t < tail:
            s = torch.full((m,), n - tail + t, device=v.device)
        else:
            s = (w * gain).masked_fill(~open_, -1.0).argmax(1)
        ws, cs = w[at, s], gain[at, s]
        u = torch.bmm(inv, v[at, s][:, :, None].contiguous())[..., 0]
        g = u * torch.sqrt(ws / (1.0 + ws * cs))[:, None]
        inv -= g[:, :, None] * g[:, None, :]
        gain = gain - torch.bmm(v, g[:, :, None].contiguous())[..., 0] ** 2
        open_[at, s] = False
        logdet += torch.log1p(ws * cs)
    return logdet


def exact(case, seed):
    c = _full(case)
    lens = _lens(c)
    L, H, G, d = c["layers"], c["kv_heads"], c["group"], c["head_dim"]
    q_all, k_all, v_all = _inputs(c, lens, seed)
    greedy = c["call"] == "greedy"
    heads = [slice(g, g + 1) for g in range(G)] if c["gqa"] == "per_head" else [slice(0, G)]
    scores = torch.zeros((L, H, sum(lens)), dtype=torch.float64, device="cuda")
    logdet = torch.zeros((len(lens), L, H), dtype=torch.float64, device="cuda")
    off = 0
    for b, n in enumerate(lens):
        step = max(1, min(L, (1 << 27) // max(1, H * n * d)))
        for l0 in range(0, L if n else 0, step):
            l1 = min(L, l0 + step)
            m = (l1 - l0) * H
            q = q_all[b, l0:l1].reshape(m, G, c["window"], d).double()
            k = k_all[l0:l1, :, off:off + n].double().reshape(m, n, d)
            v = v_all[l0:l1, :, off:off + n].double().reshape(m, n, d)
            if greedy:
                logdet[b, l0:l1] = _greedy64(c, q.reshape(m, -1, d), k, v).view(l1 - l0, H)
                continue
            total = 0.0
            for h in heads:
                total = total + _scores64(c, q[:, h].reshape(m, -1, d).contiguous(), k, v)
            scores[l0:l1, :, off:off + n] = (total / len(heads)).view(l1 - l0, H, n)
        off += n
    if greedy:
        return {"idx": None, "order": None, "logdet": logdet}
    if c["call"] == "slots":
        return {"scores": scores, "slots": None}
    return {"scores": scores, "idx": None, "k": None, "v": None}
