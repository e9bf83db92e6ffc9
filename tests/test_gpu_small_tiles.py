"""The kernels for few rows, narrow outputs and float storage where their tiles and shares can go wrong: the 64- and 128-row
tiles of the expert FFN at their edges (the shortest reduction their rings take, a split one, columns that do not
fill the last tile), the float GEMM's shared reduction with fewer units than wavefronts and with more segments than a wavefront
has lanes, on both of its tiles, the float router over remainders of its k-steps and experts, and the one-workgroup dispatch at each size where it
takes another number of steps.

Against the oracle, with the tolerances of tests/gpu_util.py; integers bit for bit.
"""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2411_16786_amd import binding as B
from paper_2411_16786_amd import workloads as WL

import gpu_util as G

pytestmark = pytest.mark.gpu

FFN_CASES = [
    # (name, rows per segment, d, F, dtype)
    ("64-row-tiles", [63, 0, 64, 65, 1, 128, 129, 40], 320, 384, "bf16"),          # first GEMM on 64 x 128 tiles
    ("four-steps", [10, 64, 70, 3], 256, 256, "bf16"),                             # the shortest ring of three stages
    ("half-last-column-tile", [100, 31, 65, 0], 576, 1088, "bf16"),                # N % 128 == 64 in both GEMMs
    ("long-reduction", [64, 127, 1, 30], 256, 2048, "bf16"),
    ("odd-steps", [64, 65, 0, 17], 256, 2112, "bf16"),                             # 33 steps of a three-stage ring
    ("128-row-tiles", [127, 128, 129, 700, 1, 0, 416, 400], 1088, 1536, "bf16"),   # second GEMM on 128 x 128, ragged columns
    ("three-shares-of-k", [64, 100, 0, 70], 1152, 4608, "bf16"),                   # second GEMM: 24 steps a share on 128 x 192
    ("first-gemm-many-rows", [500, 400], 256, 384, "bf16"),                        # full row tiles, few of them
    ("second-on-128x192", [700, 450, 513, 640, 380, 511, 300, 602], 1152, 128, "bf16"),      # two steps of a two-stage ring
    ("second-on-256x192", [1391, 612, 1204, 893, 1347, 701, 1120, 924], 1152, 192, "bf16"),  # four wavefronts, three steps
    ("f32-one-unit", [5, 33, 0, 32], 16, 16, "f32"),                               # K = 16: three of four shares are empty
    ("f32-five-units", [31, 32, 33, 64], 80, 48, "f32"),
    ("f32-many-units", [17, 65, 1, 96], 208, 400, "f32"),
    ("f32-70-segments", [1, 33, 0, 7, 32, 2, 40] * 10, 48, 80, "f32"),             # the segment table exceeds 64 lanes
    ("f32-1024-segments", [(g * 7) % 5 * (g % 3 != 1) + 70 * (g % 256 == 255) for g in range(1024)], 32, 48, "f32"),      # many of them empty
    ("f32-65-segments", [0] * 64 + [33], 16, 16, "f32"),                           # the only rows beyond the lanes' first load
    ("f32-64x64-tiles", [639, 0, 64, 65, 127, 300, 1], 48, 2704, "f32"),           # first GEMM: 43 columns of tiles, the last a quarter full
    ("f32-64x64-second", [513, 448, 1], 2576, 48, "f32"),                          # second GEMM, three units for four shares
    ("f32-64x64-70-segments", [300, 2, 64, 0, 130, 65, 200] * 10, 16, 336, "f32"), # more segments than lanes, one unit of K
]


@pytest.mark.parametrize("case", FFN_CASES, ids=[c[0] for c in FFN_CASES])
@pytest.mark.parametrize("scatter", [False, True])
def test_ffn_small_tiles(case, scatter):
    name, seg_rows, d, F, dtype = case
    print(f"\nsmall tiles {name} scatter={scatter}", flush=True)
    rows, n_seg = int(sum(seg_rows)), len(seg_rows)
    E = min(n_seg, 8)
    _, _, _, W1, b1, W2, b2 = G.small_inputs(71, 4, d, E, F, dtype, bias=True, w_std=0.02)
    r = np.random.Generator(np.random.PCG64(72))
    xp = WL.to_storage(r.standard_normal((rows, d), dtype=np.float32), dtype)
    seg_offsets = np.concatenate([[0], np.cumsum(seg_rows)]).astype(np.int32)
    seg_expert = (np.arange(n_seg) * 3 % E).astype(np.int32)
    ref = O.expert_ffn(xp, seg_offsets, seg_expert, W1, b1, W2, b2)
    ctx = B.Context(rows, d, F, E, 1, dtype)
    ws = torch.empty(ctx.workspace_bytes(), dtype=torch.uint8, device=G.DEV)
    args = (G.i32_dev(seg_offsets), G.i32_dev(seg_expert), rows, G.to_dev(W1, dtype), G.f32_dev(b1), G.to_dev(W2, dtype),
            G.f32_dev(b2))
    h = torch.full((rows + 3, d), 9.0, dtype=ctx.torch_dtype, device=G.DEV)
    if scatter:          # gathered on the way in, scattered on the way out: token perm[r] is row r's
        perm = r.permutation(rows).astype(np.int32)
        x_tok = np.empty_like(xp)
        x_tok[perm] = xp
        ctx.moe_expert_ffn_commit(G.to_dev(x_tok, dtype), G.i32_dev(perm), G.i32_dev(perm), *args, None, None, h, None, ws, T=rows)
        torch.cuda.synchronize()
        got = G.to_np(h)[perm]
    else:
        ctx.moe_expert_ffn(G.to_dev(xp, dtype), *args, h, ws)
        torch.cuda.synchronize()
        got = G.to_np(h)[:rows]
    assert (G.to_np(h)[rows:] == 9.0).all()
    if dtype == "f32":
        G.assert_close_storage(got, ref, "f32", name)
    else:
        G.assert_close_expert_rows(got, ref, name)


def test_float_ffn_bits_do_not_depend_on_the_tile():
    """The first segment alone runs on 32 x 32 tiles, with the others on 64 x 64 (first GEMM, 43 columns of tiles)."""
    seg_rows, d, F = [300, 200, 700], 48, 2704
    rows = sum(seg_rows)
    _, _, _, W1, b1, W2, b2 = G.small_inputs(77, 4, d, 3, F, "f32", bias=True, w_std=0.02)
    x = np.random.Generator(np.random.PCG64(78)).standard_normal((rows, d), dtype=np.float32)
    ctx = B.Context(rows, d, F, 3, 1, "f32")
    ws = torch.empty(ctx.workspace_bytes(), dtype=torch.uint8, device=G.DEV)
    weights = (G.to_dev(W1, "f32"), G.f32_dev(b1), G.to_dev(W2, "f32"), G.f32_dev(b2))
    h = []
    for n_seg in (3, 1):
        off = np.concatenate([[0], np.cumsum(seg_rows[:n_seg])]).astype(np.int32)
        out = torch.zeros((rows, d), device=G.DEV)
        ctx.moe_expert_ffn(G.to_dev(x, "f32"), G.i32_dev(off), G.i32_dev(np.arange(n_seg, dtype=np.int32)), int(off[-1]), *weights, out, ws)
        h.append(out[:seg_rows[0]])
    torch.cuda.synchronize()
    assert torch.equal(h[0], h[1]) and bool(h[0].any())


@pytest.mark.parametrize("d", [16, 48, 64, 80, 400, 1040, 4096])
@pytest.mark.parametrize("E,k", [(1, 1), (3, 2), (16, 3), (17, 2), (33, 4), (64, 2)])
def test_float_gate(d, E, k):
    T = 37
    print(f"\nfloat gate d={d} E={E} k={k}", flush=True)
    x, Wg, bg, *_ = G.small_inputs(73 + d + E, T, d, E, 16, "f32")
    ctx = B.Context(T, d, 16, E, k, "f32")
    scores = torch.empty((T, k), dtype=torch.float32, device=G.DEV)
    idx = torch.empty((T, k), dtype=torch.int32, device=G.DEV)
    logits = torch.empty((T, E), dtype=torch.float32, device=G.DEV)
    ctx.moe_gate(G.to_dev(x, "f32"), G.to_dev(Wg, "f32"), G.f32_dev(bg), scores, idx, None, logits)
    torch.cuda.synchronize()
    z = O.router_logits(x, Wg, bg)
    # sums of d / 4 terms and a few more additions: |error| <= (d / 4 + 8) 2^-24 sum |x w|
    bound = (d / 4 + 8) * 2.0 ** -24 * (np.abs(x).astype(np.float64) @ np.abs(Wg).astype(np.float64).T + np.abs(bg))
    assert (np.abs(G.to_np(logits) - z) <= bound + 1e-12).all()
    picked = O.topk(G.to_np(logits).astype(np.float64), k)
    np.testing.assert_array_equal(G.to_np(idx), picked)
    np.testing.assert_allclose(G.to_np(scores), O.scores(z, picked)[1], rtol=5e-5, atol=1e-9)
    # an infinite router weight reaches the logits of its expert and no other
    if E > 1:
        Wi = Wg.copy()
        Wi[1, d - 1] = np.inf
        ctx.moe_gate(G.to_dev(x, "f32"), G.to_dev(Wi, "f32"), G.f32_dev(bg), scores, idx, None, logits)
        torch.cuda.synchronize()
        zi = G.to_np(logits)
        assert (zi[:, 1] == np.where(x[:, d - 1] > 0, np.inf, -np.inf)).all()
        assert (np.abs(np.delete(zi, 1, 1) - np.delete(z, 1, 1)) <= np.delete(bound, 1, 1) + 1e-12).all()


@pytest.mark.parametrize("d,E,k,T", [
    (1024, 2, 1, 33), (1040, 1, 1, 9), (1040, 2, 2, 33), (2048, 4, 2, 1), (2064, 4, 3, 8), (4096, 4, 2, 19),   # few experts, long rows
    (1040, 4, 2, 6144), (1040, 4, 2, 6145), (1040, 2, 2, 6145),                                                # on both sides of the line
    (1040, 5, 2, 33), (448, 8, 2, 33), (1152, 8, 2, 33)])                                                      # batches of four k-steps
@pytest.mark.parametrize("renorm,n_shared", [(False, 2), (True, 0)])
def test_float_gate_long_rows(d, E, k, T, renorm, n_shared):
    print(f"\nfloat gate d={d} E={E} k={k} T={T}", flush=True)
    x, Wg, bg, *_ = G.small_inputs(76 + d + E, T, d, E, 16, "f32")
    ctx = B.Context(T, d, 16, E, k, "f32", renorm_topk=renorm, n_shared=n_shared)
    scores = torch.full((T + 1, k + n_shared), 9.0, dtype=torch.float32, device=G.DEV)
    idx = torch.full((T + 1, k + n_shared), 9, dtype=torch.int32, device=G.DEV)
    probs, logits = (torch.full((T + 1, E), 9.0, dtype=torch.float32, device=G.DEV) for _ in range(2))
    ctx.moe_gate(G.to_dev(x, "f32"), G.to_dev(Wg, "f32"), G.f32_dev(bg), scores, idx, probs, logits)
    torch.cuda.synchronize()
    z = O.router_logits(x, Wg, bg)
    got = G.to_np(logits)[:T]
    # as in test_float_gate: sums of d / 4 terms and a few more additions
    assert (np.abs(got - z) <= (d / 4 + 8) * 2.0 ** -24 * (np.abs(x).astype(np.float64) @ np.abs(Wg).astype(np.float64).T + np.abs(bg)) + 1e-12).all()
    picked = O.topk(got.astype(np.float64), k)
    np.testing.assert_array_equal(G.to_np(idx)[:T, :k], picked)
    np.testing.assert_array_equal(G.to_np(idx)[:T, k:], np.broadcast_to(E + np.arange(n_shared), (T, n_shared)))
    p, s = O.scores(z, picked, renorm_topk=renorm)
    np.testing.assert_allclose(G.to_np(scores)[:T, :k], s, rtol=5e-5, atol=1e-9)
    assert (G.to_np(scores)[:T, k:] == 1.0).all()
    np.testing.assert_allclose(G.to_np(probs)[:T], p, rtol=5e-5, atol=1e-9)
    for t in (scores, idx, probs, logits):
        assert (G.to_np(t)[T:] == 9).all()


@pytest.mark.parametrize("n_pairs", [1, 255, 256, 257, 1023, 1024, 1025, 2048, 2049, 4095, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("E,masked", [(1, False), (16, True), (64, False)])
def test_dispatch_of_one_workgroup(n_pairs, E, masked):
    r = np.random.Generator(np.random.PCG64(74 + n_pairs + E))
    idx = r.choice(E, size=(n_pairs, 1), p=WL.zipf_weights(E, 1.2)).astype(np.int32)
    mask = (r.random((n_pairs, 1)) < 0.5).astype(np.uint8) if masked else None
    ctx = B.Context(n_pairs, 64, 64, E, 1, "bf16")
    buf = B.LayerBuffers(ctx, G.DEV)
    ctx.moe_dispatch(torch.empty((n_pairs, 64), dtype=torch.bfloat16, device=G.DEV), G.i32_dev(idx),
                     None if mask is None else G.u8_dev(mask), None, buf.counts, buf.offsets, buf.perm, buf.inv, buf.workspace)
    torch.cuda.synchronize()
    counts, offsets, perm, inv = O.dispatch(idx, mask, E)
    R = perm.shape[0]
    np.testing.assert_array_equal(G.to_np(buf.counts), counts)
    np.testing.assert_array_equal(G.to_np(buf.offsets), offsets)
    np.testing.assert_array_equal(G.to_np(buf.perm)[:R], perm)
    assert (G.to_np(buf.perm)[R:] == -1).all()
    np.testing.assert_array_equal(G.to_np(buf.inv).reshape(n_pairs, 1), inv)


@pytest.mark.parametrize("world,E_loc", [(1, 1), (4, 4), (9, 7), (8, 8), (13, 5), (16, 64)])
def test_ep_segments_scan(world, E_loc):
    r = np.random.Generator(np.random.PCG64(75))
    recv = r.integers(0, 900, (world, E_loc)).astype(np.int32)
    recv[r.random(recv.shape) < 0.2] = 0
    ctx = B.Context(16, 64, 64, E_loc, 1, "bf16")
    off = torch.empty(world * E_loc + 1, dtype=torch.int32, device=G.DEV)
    exp = torch.empty(world * E_loc, dtype=torch.int32, device=G.DEV)
    ctx.moe_ep_segments(G.i32_dev(recv), off, exp)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(G.to_np(off), np.concatenate([[0], np.cumsum(recv)]))
    np.testing.assert_array_equal(G.to_np(exp), np.tile(np.arange(E_loc), world))
