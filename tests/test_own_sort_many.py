"""Layers whose first GEMM runs on the persistent kernel and sorts up to 4096 pairs itself: every buffer the layer leaves behind has the bits of
the separate calls (with a dispatch of their own; outputs where only the layer call splits the second GEMM: within the bound of
test_layer_sums.py), at the pair counts where the sort takes another group of four steps, for workgroups that come
back for rows (a piece of a leftover tile) and those that do not, for either width and for the kernel that picks it, with every
kind of mask."""
import pytest
import torch

from paper_2411_16786_amd import binding as B

import gpu_util as G
import plan_util as P
from test_layer_sums import same_outputs, separate_calls

CASES = [
    # (T, k, n_shared, d, F, E, hot expert's bias, planned first GEMM, what it runs)
    (700, 3, 0, 384, 1536, 8, 0.0, "stream192", {"halves", "rowless"}),
    (512, 2, 0, 384, 3072, 8, 0.0, "stream192", {"halves"}),                     # 1024 pairs
    (1024, 2, 0, 512, 2560, 8, 0.0, "stream192", set()),                         # 2048: a group of four steps a wavefront
    (2049, 1, 0, 512, 2560, 8, 0.0, "stream192", set()),                         # 2049: two
    (1025, 2, 0, 384, 3072, 8, 0.0, "stream192", {"leftover"}),                  # 2050
    (1365, 2, 1, 512, 2048, 15, 1.0, "stream256", {"leftover"}),                 # 4095, one shared expert
    (1821, 1, 0, 1792, 2048, 8, 0.0, "stream256", {"halves", "rowless"}),
    (2048, 2, 0, 384, 1920, 16, 0.0, "stream192", {"whole"}),                    # 4096, more than one tile a workgroup
    (2048, 2, 0, 384, 2304, 24, 0.0, "stream256", {"whole"}),
    (1972, 2, 0, 1792, 2304, 4, 4.0, "stream192", {"leftover"}),                 # the kernel that picks its width
    (2049, 2, 0, 384, 1536, 16, 3.0, "stream192", {"leftover"}),                 # 4098: dispatched
]
POLICIES = [None, (B.REFRESH_ALL, 0), (B.REFRESH_ALG4, 1), (B.REFRESH_ALG4_RANDOM, 1), (B.REFRESH_FRACTION_TOKEN, 0), (B.REFRESH_FRACTION_PAIR, 0)]


@pytest.mark.parametrize("case", CASES)
def test_the_plan(case):
    T, k, ns, d, F, E, _, planned, _ = case
    assert P.plan(True, F, d, T * (k + ns), E + ns) == planned
    assert P.sorts_pairs("bf16", T, k + ns, E + ns, d, F) == (T * (k + ns) <= 4096)
    # (the second GEMM of these two is in three shares of one tile in the layer call, of another in the separate ones)
    assert (P.plan(False, d, F, T * (k + ns), E + ns) != P.plan(False, d, F, T * (k + ns), E + ns, sums=True)) == ((T, F) in ((512, 3072), (1025, 3072)))


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_own_sort_of_many_pairs(case):
    T, k, ns, d, F, E, hot, planned, runs = case
    print(f"\nown sort {case}", flush=True)
    x, Wg, bg, *_ = G.small_inputs(53, T, d, E, 64, "bf16")
    bg[1] += hot
    gen = torch.Generator(device=G.DEV).manual_seed(7)
    normal = lambda *s: torch.randn(s, generator=gen, device=G.DEV) * 0.05
    w = (normal(E + ns, F, d).bfloat16(), normal(E + ns, F), normal(E + ns, d, F).bfloat16(), normal(E + ns, d))
    x, Wg, bg = G.to_dev(x, "bf16"), G.to_dev(Wg, "bf16"), G.f32_dev(bg)
    for entry in POLICIES:
        policy = None if entry is None else B.Policy(entry[0], step_t=entry[1], stride_n=2, n_units=T // 2)
        ctx = B.Context(T + 2, d, F, E, k, "bf16", n_shared=ns)
        a, b = (B.LayerBuffers(ctx, G.DEV, with_cache=policy is not None) for _ in range(2))
        for buf in (a, b):
            for t in (buf.scores, buf.expert_idx, buf.mask, buf.n_refresh, buf.counts, buf.offsets, buf.perm, buf.inv, buf.y, buf.h_packed):
                t.fill_(3)
            if policy is not None:
                buf.H_cache.fill_(0.5)
                buf.S_cache.fill_(0.25)
        B.moe_layer_forward(ctx, a, x, Wg, bg, *w, policy)
        separate_calls(ctx, b, x, Wg, bg, w, policy, True, policy is not None and ns == 0)
        torch.cuda.synchronize()
        rows = a.counts[: E + ns].tolist()
        items = P.stream_items(rows, list(range(E + ns)), F, int(planned[6:]))
        print(entry, rows, items, P.describe(rows, list(range(E + ns)), d, F)[0], flush=True)
        assert entry is not None or runs <= items
        for name in ("scores", "expert_idx", "mask", "n_refresh", "counts", "offsets", "perm", "inv"):
            p, q = getattr(a, name), getattr(b, name)
            assert p is None or torch.equal(p, q), (entry, name)
        same_outputs(a, b, T, F, P.plan(False, d, F, sum(rows), E + ns) == P.plan(False, d, F, sum(rows), E + ns, sums=True), entry)
        ctx.moe_expert_ffn_status(a.workspace)


@pytest.mark.gpu
def test_rows_beyond_the_bound_are_ranked_and_reported():
    T, d, F, E, k = 2048, 384, 1536, 16, 2
    x, Wg, bg, W1, b1, W2, b2 = G.small_inputs(59, T, d, E, F, "bf16")
    ctx = B.Context(T, d, F, E, k, "bf16")
    dev = [G.to_dev(x, "bf16"), G.to_dev(Wg, "bf16"), G.f32_dev(bg), G.to_dev(W1, "bf16"), G.f32_dev(b1), G.to_dev(W2, "bf16"), G.f32_dev(b2)]
    a, b = (B.LayerBuffers(ctx, G.DEV) for _ in range(2))
    for buf, rows in ((a, T * k), (b, T * k - 700)):
        buf.perm.fill_(3)
        buf.inv.fill_(3)
        B.moe_layer_forward(ctx, buf, *dev, max_rows=rows)
    for name in ("counts", "offsets", "perm", "inv"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    ctx.moe_expert_ffn_status(a.workspace)
    with pytest.raises(B.MoeError):
        ctx.moe_expert_ffn_status(b.workspace)
