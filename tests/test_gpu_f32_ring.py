"""The float expert FFN where its ring kernel is considered (K a multiple of 128, from 256 on): the shortest share of K, several tiles per workgroup, row
blocks that do not exist, columns that do not fill the last tile, empty segments, experts whose tiles spill to other XCDs, both tiles, with and
without gather, scatter and biases.  Against the oracle, with the tolerances of tests/gpu_util.py."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2411_16786_amd import binding as B
from paper_2411_16786_amd import workloads as WL

import gpu_util as G

pytestmark = pytest.mark.gpu

CASES = [
    # (name, rows per segment, d, F)
    ("two-stages", [1, 16, 17, 32, 33, 0, 64], 256, 256),            # few tiles: the other kernel
    ("two-stages-on-the-ring", [1, 16, 17, 32, 33, 0, 64], 256, 1152),
    ("three-and-five", [31, 5, 0, 40], 384, 640),
    ("ragged-columns", [33, 1, 65], 256, 272),                       # a last tile of 16 columns, but few tiles at K = 256: the other kernel (second: K = 272)
    ("ragged-columns-on-the-ring", [33, 1, 65], 384, 272),
    ("many-tiles-each", [700, 0, 30, 333], 256, 1152),               # workgroups with several 32 x 32 tiles; one expert spills
    ("one-expert-of-nine", [0] * 8 + [97], 384, 256),
    ("many-tiles-two-stages", [1000, 900, 1100, 31], 256, 2176),     # K = 256 (second: K = 2176)
    ("wide-second", [260, 255, 1, 0, 190], 1152, 1536),
    ("wide-first", [1000, 0, 900, 1100], 768, 944),                  # 64 x 64 tiles, a last one of 48 columns (second: K = 944, the other kernel)
    ("very-many-rows", [1500], 256, 10240),                          # first GEMM: 64 x 64 tiles of the other kernel
    ("64-segments", [g % 5 * 3 for g in range(64)], 256, 384),
]


@pytest.mark.parametrize("case", range(len(CASES)), ids=[c[0] for c in CASES])
@pytest.mark.parametrize("scatter,bias", [(False, True), (True, True), (True, False)])
def test_float_ffn_ring(case, scatter, bias):
    name, seg_rows, d, F = CASES[case]
    print(f"\nfloat ring {name} scatter={scatter} bias={bias}", flush=True)
    rows, n_seg = int(sum(seg_rows)), len(seg_rows)
    E = min(n_seg, 9)
    _, _, _, W1, b1, W2, b2 = G.small_inputs(171 + case, 4, d, E, F, "f32", bias=bias, w_std=0.02)
    r = np.random.Generator(np.random.PCG64(172))
    xp = r.standard_normal((rows, d), dtype=np.float32)
    seg_offsets = np.concatenate([[0], np.cumsum(seg_rows)]).astype(np.int32)
    seg_expert = (np.arange(n_seg) * 2 % E).astype(np.int32)
    ref = O.expert_ffn(xp, seg_offsets, seg_expert, W1, b1, W2, b2)
    ctx = B.Context(rows, d, F, E, 1, "f32")
    ws = torch.empty(ctx.workspace_bytes(), dtype=torch.uint8, device=G.DEV)
    args = (G.i32_dev(seg_offsets), G.i32_dev(seg_expert), rows, G.to_dev(W1, "f32"), G.f32_dev(b1), G.to_dev(W2, "f32"), G.f32_dev(b2))
    h = torch.full((rows + 3, d), 9.0, device=G.DEV)
    perm = r.permutation(rows).astype(np.int32) if scatter else np.arange(rows)
    if scatter:          # gathered on the way in, scattered on the way out: token perm[r] is row r's
        x_tok = np.empty_like(xp)
        x_tok[perm] = xp
        ctx.moe_expert_ffn_commit(G.to_dev(x_tok, "f32"), G.i32_dev(perm), G.i32_dev(perm), *args, None, None, h, None, ws, T=rows)
    else:
        ctx.moe_expert_ffn(G.to_dev(xp, "f32"), *args, h, ws)
    torch.cuda.synchronize()
    assert (G.to_np(h)[rows:] == 9.0).all()
    G.assert_close_storage(G.to_np(h)[perm], ref, "f32", name)
