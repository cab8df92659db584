"""TOP-B selection and the evicted-slot lists at the lengths where the selection
changes its path (every key in a register, sampled, staged; kept or evicted
tokens ranked; the bitmap's end), in both launch shapes, on scores with many
ties, NaN and -0: bit for bit the oracle's rule. The result is the same on every
path: which one a unit takes is counted by test_select_bracket.py."""

import numpy as np
import pytest
import torch

from oracle import jacap_oracle as jo

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jacap():
    from paper_2609_08131_amd import jacap as j
    return j


def _scores(rng, n, kind):
    if kind == "ties":
        s = rng.integers(0, 7, size=n).astype(np.float32)
        s[rng.random(n) < 0.1] = -0.0
    else:
        s = np.exp(4.0 * rng.standard_normal(n)).astype(np.float32)
    s[rng.random(n) < 0.02] = np.nan
    return s


WIDE = [1, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 8191, 8193, 16384, 16385, 65535, 65600]
NARROW = [2047, 2048, 2049, 4096, 4097, 9000]


@pytest.mark.parametrize("kind", ["ties", "spread"])
@pytest.mark.parametrize("layers,heads,lens,budget,protect", [
    (1, 2, WIDE, 700, 0),
    (1, 2, WIDE, 1, 0),
    (1, 1, WIDE, 1500, 65),       # units that keep more than half among them
    (1, 1, WIDE, 65000, 3),       # ... and one whose evicted list ends past the bitmap
    (1, 1, WIDE[:12], 8190, 0),
    (4, 64, NARROW, 257, 16),     # 1536 units: the narrow shape
    (4, 64, [2176, 2100, 2049, 1900, 2304, 2048], 2048, 5),
    # large budgets and long contexts: bands of a larger sample, kept and evicted
    (1, 1, [131072, 262145, 20000, 8192], 8192, 0),
    (1, 1, [200001, 524288], 2048, 7),
    (1, 1, [40000, 12000, 8192, 3000], 7900, 9),
    (1, 2, [40000, 131072], 36000, 0),
])
def test_paths(jacap, kind, layers, heads, lens, budget, protect):
    rng = np.random.default_rng(7)
    T, B, d = sum(lens), len(lens), 64
    z = torch.zeros((), dtype=torch.bfloat16, device="cuda")
    kv = z.expand(layers, heads, T, d).contiguous() if layers * heads * T * d < (1 << 29) else None
    if kv is None:   # only shapes and strides matter here
        kv = torch.empty((layers, heads, T, d), dtype=torch.bfloat16, device="cuda")
    q = z.expand(B, layers, heads, 1, d).contiguous()
    offs = torch.tensor(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), device="cuda")
    prob = jacap.prepare(q, kv, kv, offs, lens, jacap.Params(budget_k=budget, protect_last=protect))
    host = np.stack([_scores(rng, T, kind) for _ in range(layers * heads)]).reshape(layers, heads, T)
    scores = torch.from_numpy(host).cuda()
    jacap.select(prob.cfg, prob.batch, scores, prob.idx, prob.ws)
    slots = jacap.alloc_slots(prob, lens)
    slots.fill_(-7)
    jacap.select_evicted(prob.cfg, prob.batch, scores, slots, prob.ws)
    torch.cuda.synchronize()
    idx, ev = prob.idx.cpu().numpy(), slots.cpu().numpy()
    lo = 0
    for b, n in enumerate(lens):
        for l in range(layers):
            for h in range(heads):
                want = np.asarray(jo.select_top(host[l, h, lo:lo + n], budget, protect))
                got = idx[b, l, h]
                assert np.array_equal(got[:len(want)], want), (b, n, l, h)
                assert np.all(got[len(want):] == -1)
                gone = np.setdiff1d(np.arange(n), want)
                assert np.array_equal(ev[b, l, h][:len(gone)], gone), (b, n, l, h)
                assert np.all(ev[b, l, h][len(gone):] == -1)
        lo += n


@pytest.mark.parametrize("n,budget", [(500, 60), (3000, 700), (20000, 300)])
def test_subnormal_and_infinite_scores(jacap, n, budget):
    """Order kept below fp32's normal range, and between it, -0, the infinities and NaN."""
    rng = np.random.default_rng(n)
    s = (rng.standard_normal(n) * 1e-41).astype(np.float32)
    s[rng.random(n) < 0.05] = -0.0
    s[rng.random(n) < 0.01] = np.inf
    s[rng.random(n) < 0.01] = -np.inf
    s[rng.random(n) < 0.01] = np.nan
    z = torch.zeros((1, 1, n, 64), dtype=torch.bfloat16, device="cuda")
    offs = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    prob = jacap.prepare(z[:, :, :1].unsqueeze(0), z, z, offs, [n], jacap.Params(budget_k=budget))
    jacap.select(prob.cfg, prob.batch, torch.from_numpy(s).cuda().reshape(1, 1, n), prob.idx, prob.ws)
    torch.cuda.synchronize()
    assert np.array_equal(prob.idx.cpu().numpy()[0, 0, 0], np.asarray(jo.select_top(s, budget)))
