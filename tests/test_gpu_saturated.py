"""A centre softmax saturated so far (a gap of several hundred between the sink's
logit and the next) that the squared weights leave fp64's range: with a ridge the
scores are zero in fp32, finite and unflagged, whatever the chunks that the logits
fall into; the greedy selection's objective is that of the ridge alone."""

import math

import numpy as np
import pytest
import torch

from jacap_synth import make_case
from helpers import gpu_unit_scores, oracle_unit, run_gpu, score_errors, tol_for, unit_list

pytestmark = pytest.mark.gpu


def _case(n, d, dtype, seqs=1):
    return make_case("ragged16", seq_lens=[n] * seqs, num_layers=1, num_kv_heads=2, num_q_heads=4,
                     head_dim=d, window=8, dtype=dtype).to("cuda")


# one K-pass chunk of a small batch, several, several of 1024 tokens; enough
# sequences for chunks of 1024 tokens
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64)])
@pytest.mark.parametrize("n,seqs", [(200, 1), (1000, 1), (5000, 1), (1100, 300)])
@pytest.mark.parametrize("gap", [140.0, 170.0, 250.0, 340.0])
def test_ridge_zero(dtype, d, n, seqs, gap):
    """Without a ridge the scores do not depend on the weights' scale: one token's logit
    `gap` above those of otherwise plain keys leaves them what the oracle computes."""
    case = _case(n, d, dtype, seqs)
    gen = torch.Generator(device="cuda").manual_seed(3)
    case.k.copy_(torch.randn(case.k.shape, generator=gen, device="cuda"))
    for b in range(seqs):
        mu = case.q_win[b, 0].float().reshape(2, -1, d).mean(1)      # per KV head
        case.k[0, :, b * n + 7] = (mu * (gap * math.sqrt(d) / (mu * mu).sum(1, keepdim=True))).to(case.k.dtype)
    prob, flags = run_gpu(case, 16, tau=1.0, ridge=0.0)
    assert flags == 0
    for b, l, h in unit_list(case)[:6]:
        o = oracle_unit(case, b, l, h, 16, tau=1.0, ridge=0.0)
        err = score_errors(gpu_unit_scores(case, prob, b, l, h), o["scores"])
        assert err.max() <= tol_for(case), (b, h, float(err.max()))


@pytest.mark.parametrize("n", [300, 5000])
def test_matrix_ridge(n):
    case = _case(n, 128, "bf16")
    R = np.stack([np.eye(128) * 2.0] * 2)[None]
    prob, flags = run_gpu(case, 16, tau=0.05, ridge_matrices=R)
    assert flags == 0 and bool(torch.isfinite(prob.scores).all())


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("n", [300, 1100, 13000])
def test_greedy_objective_stays_finite(dtype, n):
    from paper_2609_08131_amd import jacap
    case = _case(n, 64, dtype)
    for tau in (0.05, 0.01):
        prob = jacap.prepare_greedy(case.q_win, case.k, case.v, case.seq_offsets, case.seq_lens,
                                    jacap.Params(budget_k=12, temperature=tau, ridge=2.0))
        jacap.run_greedy(prob, case.q_win, case.k, case.v)
        assert jacap.read_status(prob.ws) == 0
        want = 64 * math.log(2.0)
        assert np.allclose(prob.logdet.cpu().numpy(), want, rtol=1e-9), tau
        for h in range(2):
            picks = prob.order[0, 0, h].cpu().numpy()
            assert len(set(picks.tolist())) == 12 and picks.min() >= 0 and picks.max() < n
