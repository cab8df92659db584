"""fp32 batches of unequal sequences, whose fp64 Gram partials are placed by tokens:
lengths that end at and around chunk borders, sequences that start anywhere in a
chunk, pooled and per query head; every unit against the oracle."""

import pytest

from jacap_synth import make_case

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
