"""The persistent grouped GEMM of the expert FFN (ffn_stream.hpp) where its work lists can go wrong: whole rounds
followed by leftover tiles that are run whole, as halves or as quarters (among them pieces without rows or without
columns), ragged and empty segments, a hot expert whose tiles spill over to other XCDs, the shortest reduction the rings
take, and more than 64 tiles per workgroup (the places of the tiles are looked up 64 at a time).

Against the oracle on sampled rows; tolerances of the bf16 expert FFN (tests/gpu_util.py).
"""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2411_16786_amd import binding as B
from paper_2411_16786_amd import workloads as WL

import gpu_util as G

pytestmark = pytest.mark.gpu

CASES = [
    # (name, rows per segment, d, F, what the first and the second GEMM run: asserted by tests/test_ffn_plan.py)
    ("halves-of-192", [1280, 1025, 1150, 1281, 1, 0, 2300, 1290], 1792, 512, "stream192 halves rowless",
     "stream192 halves rowless whole"),
    ("quarters-without-rows", [300, 257, 384, 129, 640, 511, 128, 385], 1152, 4608, "stream256 quarters rowless whole", "128x192deep"),
    ("halves-of-256", [241, 459, 194, 99, 481, 1021, 211, 237], 576, 3072, "stream256 halves leftover", "64x128"),
    ("quarters-without-columns", [524, 656, 1414, 1026, 822, 358, 411, 703, 231], 384, 2176,
     "stream256 columnless leftover quarters whole", "128x192deep/2"),
    ("second-halves-of-192", [266, 772, 1415, 446, 260, 793, 564], 2176, 512, "64x128", "stream192 halves leftover rowless whole"),
    ("second-quarters-without-columns", [1437, 787, 983, 1318, 2394, 1359, 506, 1054, 2086], 1152, 384, "stream192 halves rowless",
     "stream256 columnless leftover quarters rowless whole"),
    ("second-halves-of-256", [654, 1625, 1068, 1508, 1235, 1873, 1025, 1028], 2176, 384, "64x128",
     "stream256 halves leftover rowless whole"),
    ("leftover-run-whole", [700, 900, 650, 1100, 820, 760, 905, 1024], 1152, 4608, "stream192 leftover whole", "256x192w4"),
    ("hot-expert", [6000, 30, 0, 200, 61, 90, 263, 1500], 1152, 1536, "stream256 leftover", "256x192w4"),
    ("columns-not-a-multiple", [520, 700, 513, 300, 1000, 800, 257, 400], 1088, 1600, "stream192 leftover", "128x192deep"),
    ("six-steps", [1391, 612, 1204, 893, 1347, 701, 1120, 924], 384, 4608, "stream256 leftover whole", "128x128"),
    ("more-than-64-tiles-each", [16384 - 77], 384, 66560, "stream256 many whole", "128x192deep"),
]


def segment_experts(E):
    return np.roll(np.arange(E, dtype=np.int32), 1)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_persistent_ffn_on_sampled_rows(case):
    name, seg_rows, d, F = case[:4]
    E, rows = len(seg_rows), int(sum(seg_rows))
    print(f"\nstream ffn {name}", flush=True)
    _, _, _, W1, b1, W2, b2 = G.small_inputs(61, 4, d, E, F, "bf16", bias=True, w_std=0.02 if F < 10000 else 0.005)
    r = np.random.Generator(np.random.PCG64(62))
    xp = WL.to_storage(r.standard_normal((rows, d), dtype=np.float32), "bf16")
    seg_offsets = np.concatenate([[0], np.cumsum(seg_rows)]).astype(np.int32)
    seg_expert = segment_experts(E)
    ctx = B.Context(rows + 8, d, F, E, 1, "bf16")
    h = torch.full((rows + 8, d), 9.0, dtype=torch.bfloat16, device=G.DEV)
    ws = torch.empty(ctx.workspace_bytes(), dtype=torch.uint8, device=G.DEV)
    x_dev = G.to_dev(xp, "bf16")
    args = (G.i32_dev(seg_offsets), G.i32_dev(seg_expert), rows, G.to_dev(W1, "bf16"), G.f32_dev(b1), G.to_dev(W2, "bf16"),
            G.f32_dev(b2))
    ctx.moe_expert_ffn(x_dev, *args, h, ws)
    torch.cuda.synchronize()
    got = G.to_np(h)
    edge = []
    for g in range(E):
        lo, hi = int(seg_offsets[g]), int(seg_offsets[g + 1])
        edge += [q for q in (lo, lo + 127, lo + 128, lo + 255, lo + 256, hi - 1) if lo <= q < hi]
    sel = np.unique(np.concatenate([np.array(edge, np.int64), r.integers(0, rows, 60 if F < 10000 else 12)])).astype(np.int32)
    ref = O.expert_ffn(xp, seg_offsets, seg_expert, W1, b1, W2, b2, rows_sel=sel)
    G.assert_close_expert_rows(got[sel], ref, name)
    assert (got[rows:] == 9.0).all()                                   # rows outside every segment are left untouched
    assert np.isfinite(got[:rows]).all() and (got[:rows] != 9.0).any(axis=1).all()
    # gathered rows in another order of tokens: the same bits row for row
    perm = r.permutation(rows).astype(np.int32)
    x_tok = torch.empty_like(x_dev)
    x_tok[torch.from_numpy(perm).long().to(G.DEV)] = x_dev
    h2 = torch.full_like(h, 7.0)
    ctx.moe_expert_ffn_rows(x_tok, G.i32_dev(perm), *args, h2, ws)
    torch.cuda.synchronize()
    assert torch.equal(h2[:rows], h[:rows])
    # ... and scattered on the way out
    pairs = r.permutation(rows + 8)[:rows].astype(np.int32)
    h3 = torch.full_like(h, 5.0)
    ctx.moe_expert_ffn_commit(x_tok, G.i32_dev(perm), G.i32_dev(pairs), *args, None, None, h3, None, ws, T=rows + 8)
    torch.cuda.synchronize()
    where = torch.from_numpy(pairs).long().to(G.DEV)
    assert torch.equal(h3[where], h[:rows])
    h3[where] = 5.0
    assert bool((h3 == 5.0).all())
