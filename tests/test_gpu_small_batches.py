"""Batches that do not fill the chip: K-pass chunks of 256 tokens (their statistics
held in a later pass's buffer) and weight chunks down to 1024 tokens, at the
lengths where these end, against the oracle at the stated tolerances."""

import pytest

from jacap_synth import make_case

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
