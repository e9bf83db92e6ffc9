"""The persistent GEMM takes the other tile width where the real segment sizes say so: cases in either direction for either GEMM (that they
do is checked on the CPU), against the oracle on sampled rows, gathered and scattered rows bit for bit."""
import pytest

import plan_util as P
import test_gpu_ffn_stream as stream

CASES = [
    # (name, rows per segment, d, F, planned on the estimate, what the kernel runs)
    ("first-to-192", [1931, 595], 1792, 6144, ("stream256", "128x192deep"), ("stream192 halves rowless whole", "128x192deep")),
    ("first-to-256", [3944, 746, 512, 1483], 1792, 2304, ("stream192", "stream256"), ("stream256 leftover", "stream256 leftover")),
    ("second-to-256", [256, 1485, 1449, 1, 256, 1777, 936, 2330], 1792, 2304, ("stream192", "stream192"),
     ("stream192 leftover whole", "stream256 leftover whole")),
    ("second-to-192", [498, 4841], 2304, 4608, ("stream192", "stream256"), ("stream192 leftover whole", "stream192 leftover whole")),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_the_width_changes(case):
    name, seg_rows, d, F, planned, taken = case
    assert P.ffn_plans(sum(seg_rows), len(seg_rows), d, F) == planned
    # (the kernel's experts are rolled by one against the segments, which deals the tiles to other XCDs but changes no number of them)
    assert P.describe(seg_rows, list(range(len(seg_rows))), d, F) == taken


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_either_width_against_the_oracle(case):
    stream.test_persistent_ffn_on_sampled_rows(case)
