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
    # (name, rows per segment, d, F): tiles per XCD of the two GEMMs on 256 rows x 256 (192) columns
    ("one-round-and-quarters", [1280, 1025, 1150, 1281, 1, 0, 2300, 1290], 1792, 512),
    ("halves-with-empty-lower-half", [300, 257, 384, 129, 640, 511, 128, 385], 1152, 4608),
    ("leftover-run-whole", [700, 900, 650, 1100, 820, 760, 905, 1024], 1152, 4608),
    ("hot-expert", [6000, 30, 0, 200, 61, 90, 263, 1500], 1152, 1536),
    ("columns-not-a-multiple", [520, 700, 513, 300, 1000, 800, 257, 400], 1088, 1600),
    ("six-steps", [1391, 612, 1204, 893, 1347, 701, 1120, 924], 384, 4608),
    ("more-than-64-tiles-each", [16384 - 77], 384, 66560),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_persistent_ffn_on_sampled_rows(case):
    name, seg_rows, d, F = case
    E, rows = len(seg_rows), int(sum(seg_rows))
    print(f"\nstream ffn {name}", flush=True)
    _, _, _, W1, b1, W2, b2 = G.small_inputs(61, 4, d, E, F, "bf16", bias=True, w_std=0.02 if F < 10000 else 0.005)
    r = np.random.Generator(np.random.PCG64(62))
    xp = WL.to_storage(r.standard_normal((rows, d), dtype=np.float32), "bf16")
    seg_offsets = np.concatenate([[0], np.cumsum(seg_rows)]).astype(np.int32)
    seg_expert = np.roll(np.arange(E, dtype=np.int32), 1)
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
