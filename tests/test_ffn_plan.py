"""The tile rule of the expert FFN on the CPU: the cases of the GPU tests run what they are named for, and between them every tile and
every kind of work item that the rule can lead to."""
import itertools

import pytest

import plan_util as P
import test_gpu_f32_ring as ring
import test_gpu_ffn_stream as stream
import test_gpu_parity as parity
import test_gpu_small_tiles as small

SMALL_TILES = {      # bf16 cases of test_gpu_small_tiles.py: tiles of the first and the second GEMM
    "64-row-tiles": ("64x128", "staged"),
    "four-steps": ("64x128", "64x128"),
    "half-last-column-tile": ("64x128", "64x128"),
    "long-reduction": ("64x128", "64x128"),
    "odd-steps": ("64x128", "64x128"),
    "128-row-tiles": ("stream192", "128x128"),
    "three-shares-of-k": ("128x192deep", "128x192deep/3"),
    "first-gemm-many-rows": ("64x128", "64x128"),
    "second-on-128x192": ("64x128", "128x192"),
    "second-on-256x192": ("128x192deep", "256x192"),
}


@pytest.mark.parametrize("case", stream.CASES, ids=[c[0] for c in stream.CASES])
def test_persistent_cases_run_what_they_say(case):
    name, seg_rows, d, F, first, second = case
    assert P.describe(seg_rows, stream.segment_experts(len(seg_rows)), d, F) == (first, second)


def test_small_cases_run_what_they_say():
    got = {c[0]: P.ffn_plans(sum(c[1]), len(c[1]), c[2], c[3]) for c in small.FFN_CASES if c[4] == "bf16"}
    assert got == SMALL_TILES


WIDE_TILES = {       # of test_gpu_parity.py
    "xl-8192-rows": ("stream256", "256x192w4"), "xl-4096-rows": ("stream192", "128x192deep"),
    "xl-2048-rows": ("stream256", "128x192deep/2"), "xl-700-rows": ("128x192deep", "128x192deep/3"),
    "k-64": ("128x192", "staged"), "k-128": ("128x192", "64x128"), "k-192": ("128x192", "staged"), "k-256": ("128x192deep", "64x128"),
    "k-256-few-rows": ("128x192deep", "64x128"),
    "k2-320": ("staged", "256x192w4"), "k2-384": ("64x128", "256x192w4"), "k2-256": ("64x128", "256x192w3"),
}


def test_wide_cases_run_what_they_say():
    got = {c[0]: P.ffn_plans(sum(c[1]), len(c[1]), c[2], c[3]) for c in parity.WIDE_FFN_CASES}
    assert {name: got[name] for name in WIDE_TILES} == WIDE_TILES


def test_every_kind_of_persistent_item_is_run_by_either_gemm():
    seen = {(gemm, line.split()[0], item) for c in stream.CASES for gemm, line in enumerate(c[4:]) for item in line.split()[1:]}
    for gemm, (tile, items) in itertools.product((0, 1), (("stream192", "whole leftover halves rowless"),
                                                          ("stream256", "whole leftover halves quarters rowless columnless"))):
        for item in items.split():
            assert (gemm, tile, item) in seen


def test_every_tile_of_the_rule_is_run_by_a_case():
    widths = [64, 128, 192, 256, 320, 384, 448, 576, 768, 1024, 1152, 1536, 1792, 2048, 4608, 7168, 8192]
    rows = [int(2.0 ** (i / 2)) for i in range(0, 36)]
    reached = set()
    for d, F, n_seg, R, experts in itertools.product(widths, widths, (1, 2, 4, 8, 16, 32, 64, 80), rows, (2, 64)):
        first, second = P.ffn_plans(R, n_seg, d, F, experts)
        reached |= {(0, first), (1, second)}
    run = set()
    cases = stream.CASES + [c for c in small.FFN_CASES if c[4] == "bf16"] + parity.WIDE_FFN_CASES
    for c in cases:
        first, second = P.ffn_plans(sum(c[1]), len(c[1]), c[2], c[3])
        run |= {(0, first), (1, second)}
    assert reached <= run, sorted(reached - run)


@pytest.mark.parametrize("gelu,N,K,rows,n_seg,n_experts,tile", [
    # second GEMM of a few experts: three shares of K while they run in one round and the second pass is short
    (False, 2048, 8192, 500, 2, 2, "128x192deep/3"), (False, 1152, 4608, 968, 2, 2, "128x192deep/3"), (False, 1152, 4608, 1219, 2, 2, "64x128"),
    (False, 1152, 4608, 900, 8, 8, "64x128"),
    # many experts with few rows each: a tile for every one of them
    (False, 1152, 4608, 960, 32, 32, "128x192deep"), (False, 1152, 4608, 960, 32, 4, "128x192deep"), (False, 640, 2560, 768, 64, 8, "64x128"),
    # first GEMM in several rounds: small tiles only where cold weights are what the time goes to
    (True, 7168, 1792, 1024, 16, 16, "64x128"), (True, 7168, 1792, 1900, 16, 16, "128x192"), (True, 2048, 512, 4864, 64, 64, "128x192"),
    (True, 4096, 1024, 1536, 32, 32, "64x128"), (True, 4096, 1024, 4608, 64, 64, "128x192"),
    (True, 4608, 1152, 992, 16, 4, "128x192"),
    # ... or in whole rounds
    (True, 4096, 1024, 768, 32, 8, "64x128"), (True, 4608, 1152, 1280, 64, 8, "128x192"), (True, 1536, 384, 1024, 64, 64, "128x192"),
])
def test_lines_between_the_small_tiles(gelu, N, K, rows, n_seg, n_experts, tile):
    assert P.plan(gelu, N, K, rows, n_seg, n_experts) == tile


@pytest.mark.parametrize("rows,segs,d,F,tiles", [
    # either end of the ring at K = 256, and reductions and tables that it does not take
    (64, 4, 64, 256, ("direct32", "direct32")), (861, 8, 256, 256, ("direct32", "direct32")), (1448, 8, 256, 256, ("ring32", "ring32")),
    (11585, 4, 256, 768, ("ring32", "ring64")), (23170, 4, 256, 1024, ("direct64", "ring64")), (11585, 32, 512, 2048, ("ring32", "ring64")),
    (300, 65, 384, 1536, ("direct32", "direct32")), (500, 8, 272, 800, ("direct32", "direct32")),
    # 64 x 64 tiles only where rows and rounds are filled
    (192, 64, 512, 2048, ("ring32", "ring32")), (1000, 64, 512, 2048, ("ring32", "ring32")), (512, 32, 768, 3072, ("ring32", "ring32")),
    (2435, 16, 384, 1536, ("ring32", "ring32")), (4096, 16, 384, 1536, ("ring32", "ring64")), (2435, 8, 384, 1536, ("ring32", "ring64")),
    (1448, 8, 512, 2048, ("ring32", "ring64")), (2435, 8, 512, 2048, ("ring32", "ring32")), (11585, 8, 768, 3072, ("ring64", "ring64")),
    (864, 8, 1152, 4608, ("ring32", "ring32")), (1448, 8, 1152, 4608, ("ring32", "ring64")), (1000, 16, 384, 1536, ("ring32", "ring32")),
    (2000, 16, 384, 1536, ("ring32", "ring64")), (1000, 8, 768, 3072, ("ring32", "ring64")), (2000, 8, 1152, 4608, ("ring64", "ring64")),
    (800, 2, 2048, 8192, ("ring64", "ring64")),
])
def test_float_tiles(rows, segs, d, F, tiles):
    assert P.f32_plans(rows, segs, d, F) == tiles


def test_float_cases_run_what_they_are_named_for():
    plans = {name: P.f32_plans(sum(seg), len(seg), d, F) for name, seg, d, F in ring.CASES}
    assert plans["two-stages-on-the-ring"][0] == plans["many-tiles-two-stages"][0] == plans["64-segments"][0] == "ring32"        # K = 256
    assert plans["ragged-columns-on-the-ring"][0] == plans["three-and-five"][0] == plans["one-expert-of-nine"][0] == "ring32"   # K = 384
    assert plans["wide-first"][0] == plans["wide-second"][1] == "ring64"
    assert plans["two-stages"] == ("direct32", "direct32") and plans["very-many-rows"][0] == "direct64"
