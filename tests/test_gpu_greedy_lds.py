"""The greedy selection's LDS kernel where it can go wrong: blocks of 256 positions
that end, pick counts around the 64 held in registers, more refreshes per pick
than it remembers (small ridge), protected tails, and the lengths at which units
stop fitting in LDS; each path replayed through the fp64 oracle (the checks and
tolerances of test_gpu_greedy.py); calls of different lengths from several host
threads at once."""

import threading

import pytest
import torch

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


def test_lengths_from_several_threads(jacap):  # noqa: F811
    problems = []
    for n, budget in ((300, 24), (11000, 24)):
        case = make_case("ragged16", seq_lens=[n], num_layers=1, num_kv_heads=2, num_q_heads=4,
                         head_dim=64, window=8, dtype="bf16").to("cuda")
        prob = jacap.prepare_greedy(case.q_win, case.k, case.v, case.seq_offsets, case.seq_lens,
                                    jacap.Params(budget_k=budget))
        jacap.run_greedy(prob, case.q_win, case.k, case.v)
        torch.cuda.synchronize()
        problems.append((case, prob, torch.cuda.Stream(), prob.order.clone()))
        prob.order.fill_(-7)
    errors = []

    def work(case, prob, stream):
        try:
            for _ in range(20):
                jacap.run_greedy(prob, case.q_win, case.k, case.v, stream)
        except Exception as e:   # noqa: BLE001 (reported by the main thread)
            errors.append(e)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(c, p, s)) for c, p, s, _ in problems]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors
    for _, prob, _, want in problems:
        assert torch.equal(prob.order, want)
