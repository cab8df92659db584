"""The fp64 path (Gram and leverage products on the fp64 MFMA) at the sizes where
its tiles end: every unit of fp32 inputs, the marked units of bf16 inputs, from
few marked units of a batch to all of them. Tolerance: the stated one of the
scores (fp32 1e-5, bf16 1e-3); bf16 units on this path are held to 5e-5, since
their products and sums are fp64 and only the weights round (their K pass sums
in fp32)."""

import numpy as np
import pytest
import torch

from jacap_synth import make_case

from helpers import BF16_TOL, FP32_TOL, gpu_unit_scores, oracle_unit, run_gpu, score_errors, unit_list

pytestmark = pytest.mark.gpu

# The workspace's per-unit flags and the one of the fp64 path (both are pinned by
# the host driver, tests/sanitize/host_driver.cpp).
FLAGS_AT, MARKED = 256, 1 << 8
MARKED_TOL = 5e-5


def _marked_units(prob, units):
    flags = prob.ws[FLAGS_AT:FLAGS_AT + 4 * units].view(torch.int32).cpu().numpy()
    return (flags & MARKED) != 0


# lens around the Gram's turns (64 tokens) and chunks (128 up), the leverage trip
# (128 tokens) and its 16-token tiles
EDGES = [130, 143, 144, 145, 255, 257, 383, 385, 512, 1025, 2177]


@pytest.mark.parametrize("dtype,d,token_major", [("fp32", 128, False), ("fp32", 64, True),
                                                 ("bf16", 128, True), ("bf16", 64, False)])
def test_every_unit_at_tile_edges(dtype, d, token_major):
    case = make_case("ragged16", seq_lens=EDGES, num_layers=1, num_kv_heads=2, num_q_heads=4,
                     head_dim=d, window=8, dtype=dtype).to("cuda")
    if token_major:   # K and V stored [L][T][H][d], passed as views
        case.k = case.k.transpose(1, 2).contiguous().transpose(1, 2)
        case.v = case.v.transpose(1, 2).contiguous().transpose(1, 2)
    # ridge 0 sends the bf16 units to the fp64 path
    prob, flags = run_gpu(case, 64, ridge=0.0 if dtype == "bf16" else 1.0)
    assert flags == 0
    units = unit_list(case)
    if dtype == "bf16":
        assert _marked_units(prob, len(units)).sum() >= len(units) // 2
    marked = _marked_units(prob, len(units)) if dtype == "bf16" else np.ones(len(units), bool)
    for i, (b, l, h) in enumerate(units):
        o = oracle_unit(case, b, l, h, 64, ridge=0.0 if dtype == "bf16" else 1.0)
        err = score_errors(gpu_unit_scores(case, prob, b, l, h), o["scores"])
        assert err.max() <= (FP32_TOL if dtype == "fp32" else BF16_TOL), (b, l, h, float(err.max()))
        if dtype == "bf16" and marked[i]:
            assert err.max() <= MARKED_TOL, (b, l, h, float(err.max()))


@pytest.mark.parametrize("d", [128, 64])
def test_few_marked_units_of_a_large_batch(d):
    """More units than compute units, of which a part take the fp64 path: the
    planted ones (one value channel scaled by 2^15, an eigenvalue of A far above the ridge) and
    the short units that are so by themselves."""
    lens = [300] * 39 + [1500]
    case = make_case("ragged16", seq_lens=lens, num_layers=2, num_kv_heads=4, num_q_heads=8,
                     head_dim=d, window=8, dtype="bf16").to("cuda")
    lo = sum(lens[:-1])
    case.v[1, 2:, lo:, 5] *= 2.0 ** 15   # two units of the last sequence
    case.v[0, 0, 300:600, 5] *= 2.0 ** 15
    prob, flags = run_gpu(case, 32, ridge=1.0)
    assert flags == 0
    units = unit_list(case)
    marked = _marked_units(prob, len(units))
    assert 3 <= marked.sum() <= len(units) // 2
    assert all(marked[units.index(x)] for x in [(39, 1, 2), (39, 1, 3), (1, 0, 0)])
    for i, (b, l, h) in enumerate(units):
        if not marked[i] and (b, l, h) not in [(39, 0, 0), (5, 1, 1)]:
            continue
        o = oracle_unit(case, b, l, h, 32, ridge=1.0)
        err = score_errors(gpu_unit_scores(case, prob, b, l, h), o["scores"])
        assert err.max() <= (MARKED_TOL if marked[i] else BF16_TOL), (b, l, h, float(err.max()))
    again, _ = run_gpu(case, 32, ridge=1.0)   # the list's order does not show
    assert torch.equal(again.scores, prob.scores)
