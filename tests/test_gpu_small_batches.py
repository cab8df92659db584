"""Batches that do not fill the chip: K-pass chunks of 256 tokens (their statistics
held in a later pass's buffer) and weight chunks down to 1024 tokens, at the
lengths where these end, against the oracle at the stated tolerances."""

import pytest

from jacap_synth import make_case

from helpers import gpu_unit_scores, oracle_unit, score_errors, tol_for, unit_list
from test_gpu_greedy import check_greedy
from test_gpu_parity import check_case, jacap  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu

EDGES = [1, 127, 128, 129, 255, 256, 257, 511, 513, 1023, 1025, 4095, 4097]


@pytest.mark.parametrize("dtype,d,window", [("bf16", 128, 130), ("bf16", 64, 7),
                                            ("fp32", 128, 33), ("fp32", 64, 16)])
def test_chunk_edges(jacap, dtype, d, window):  # noqa: F811
    # windows of fewer and of more rows than the statistics pass holds in registers
    case = make_case("ragged16", seq_lens=EDGES, num_layers=1, num_kv_heads=2, num_q_heads=4,
                     head_dim=d, window=window, dtype=dtype).to("cuda")
    check_case(case, 48, 1.0, "diag", label=f"small {dtype} d={d} w={window}", jacap=jacap)


def test_greedy_with_many_empty_sequences(jacap):  # noqa: F811
    # the chunk statistics of 301 sequences do not fit the buffer that one
    # sequence's tokens size: the K pass keeps its own
    case = make_case("ragged16", seq_lens=[0] * 300 + [4000], num_layers=1, num_kv_heads=1,
                     num_q_heads=2, head_dim=64, window=8, dtype="bf16").to("cuda")
    check_greedy(jacap, case, 24, units=[(0, 0, 0), (300, 0, 0)], label="empty sequences")


@pytest.mark.parametrize("dtype,gqa", [("bf16", "pooled"), ("bf16", "per_head"), ("fp32", "pooled"),
                                       ("fp32", "per_head")])
def test_many_short_sequences_and_a_long_one(jacap, dtype, gqa):  # noqa: F811
    # chunk counts that are multiples of 8, spread over the XCDs by one empty chunk
    case = make_case("ragged16", seq_lens=[17] * 20 + [8000, 0, 300], num_layers=1, num_kv_heads=2,
                     num_q_heads=4, head_dim=64, window=8, dtype=dtype).to("cuda")
    check_case(case, 16, 1.0, "diag", label=f"short and long {dtype} {gqa}", jacap=jacap, gqa=gqa)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_declared_length_above_the_real_ones(jacap, dtype):  # noqa: F811
    case = make_case("ragged16", seq_lens=[700, 1024, 3], num_layers=1, num_kv_heads=2, num_q_heads=4,
                     head_dim=128, window=8, dtype=dtype).to("cuda")
    prob = jacap.prepare(case.q_win, case.k, case.v, case.seq_offsets, case.seq_lens,
                         jacap.Params(budget_k=32))
    prob.batch.max_seq_len = 131072
    prob.ws = jacap.alloc_workspace(prob.cfg, prob.batch)
    jacap.run_evict(prob, case.q_win, case.k, case.v)
    assert jacap.read_status(prob.ws) == 0
    for b, l, h in unit_list(case):
        o = oracle_unit(case, b, l, h, 32)
        err = score_errors(gpu_unit_scores(case, prob, b, l, h), o["scores"])
        assert err.max() <= tol_for(case), (b, l, h, float(err.max()))
