"""The greedy selection's LDS kernel where it can go wrong: blocks of 256 positions
that end, pick counts around the 64 held in registers, more refreshes per pick
than it remembers (small ridge), protected tails, and the lengths at which units
stop fitting in LDS; each path replayed through the fp64 oracle (the checks and
tolerances of test_gpu_greedy.py)."""

import pytest

from jacap_synth import make_case

from test_gpu_greedy import check_greedy, jacap  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,budget,ridge,dtype,d,protect", [
    (256, 64, 1.0, "bf16", 128, 0),
    (257, 65, 1.0, "fp32", 128, 3),
    (255, 255, 1.0, "bf16", 64, 0),       # everything is taken
    (1025, 129, 2.0 ** -20, "fp32", 64, 65),
    (3000, 60, 2.0 ** -20, "bf16", 128, 0),   # over 64 refreshes per pick
    (12032, 20, 1.0, "bf16", 128, 0),     # the most that fit
    (12033, 20, 1.0, "bf16", 128, 0),     # one more: the kernel for long units
])
def test_greedy_lds_edges(jacap, n, budget, ridge, dtype, d, protect):  # noqa: F811
    case = make_case("ragged16", seq_lens=[n], num_layers=1, num_kv_heads=2, num_q_heads=4,
                     head_dim=d, window=8, dtype=dtype).to("cuda")
    check_greedy(jacap, case, budget, ridge=ridge, protect_last=protect,
                 label=f"lds n={n} ridge={ridge:g}")
