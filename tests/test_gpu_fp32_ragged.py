"""fp32 batches of unequal sequences (fp64 Gram, chunks cut for the longest one):
lengths that end at and around chunk borders, sequences that start anywhere in a
chunk, pooled and per query head; every unit against the oracle. Sequences with
inconsistent offsets among them leave the others' scores as they are."""

import pytest
import torch

from jacap_synth import make_case
from oracle import jacap_oracle as jo
from helpers import FP32_TOL, score_errors
from test_gpu_parity import check_case, jacap  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,heads,d,gqa", [
    ([1, 700, 0, 129, 2500, 64, 1, 1], 2, 128, "pooled"),
    ([5000, 3, 3, 3, 127, 128, 129], 1, 64, "pooled"),
    ([300] * 20 + [4097], 2, 64, "per_head"),
    ([17] * 300 + [1000], 1, 64, "pooled"),      # more sequences than partials
])
def test_unequal_fp32_sequences(jacap, lens, heads, d, gqa):  # noqa: F811
    case = make_case("ragged16", seq_lens=lens, num_layers=1, num_kv_heads=heads,
                     num_q_heads=2 * heads, head_dim=d, window=8, dtype="fp32").to("cuda")
    check_case(case, 32, 1.0, "diag", label=f"fp32 ragged {len(lens)} seqs", jacap=jacap, gqa=gqa)


@pytest.mark.parametrize("heads,d", [(1, 128), (2, 64)])
def test_valid_sequences_beside_bad_offsets(jacap, heads, d):  # noqa: F811
    """Sequences 1 and 3 are consistent and share no token, but lie in descending
    order (0 is longer than max_seq_len, 2 descends, the rest are empty): the
    flag is raised and both are scored as they are alone."""
    n, lens = 3000, [20000, 3000] + [0] * 14
    case = make_case("ragged16", seq_lens=lens, num_layers=1, num_kv_heads=heads,
                     num_q_heads=2 * heads, head_dim=d, window=8, dtype="fp32").to("cuda")
    prob = jacap.prepare(case.q_win, case.k, case.v, case.seq_offsets, case.seq_lens,
                         jacap.Params(budget_k=32))
    offs = torch.tensor([0, 20000, 23000, 17000, 20000] + [20000] * 12, dtype=torch.int32, device="cuda")
    prob.batch.seq_offsets = offs.data_ptr()
    prob.batch.max_seq_len = n
    prob.ws = jacap.alloc_workspace(prob.cfg, prob.batch)
    jacap.run_evict(prob, case.q_win, case.k, case.v)
    assert jacap.read_status(prob.ws) == jacap.FLAG_BAD_OFFSETS
    for b, t0 in ((1, 20000), (3, 17000)):
        for h in range(heads):
            # the oracle on those tokens with sequence b's window
            q = case.q_win[b, 0, 2 * h:2 * h + 2].double().cpu().numpy()
            k = case.k[0, h, t0:t0 + n].double().cpu().numpy()
            v = case.v[0, h, t0:t0 + n].double().cpu().numpy()
            o = jo.evict_unit(q, k, v, 32, tau=10.0, ridge=1.0)
            got = prob.scores[0, h, t0:t0 + n].double().cpu().numpy()
            assert score_errors(got, o["scores"]).max() <= FP32_TOL, (b, h)
    for b in (0, 2, 4):
        assert torch.all(prob.idx[b] == -1)
