"""A layer whose second GEMM is split over K: its combine adds the float shares itself.  Same bits as the separate entry points (whose
second pass adds them) where these split as well, in every buffer the layer leaves behind, for two and three shares, one to four slots,
widths that do not fill the last wavefront, biases or none, and rows that go to the packed buffer, to the cache, or to both.  Where only the
layer call splits, the sums are formed in another order: two sums of F products with chains of F / 16 additions differ by
(F / 16) 2^-24 times the sum of the products' magnitudes (about 0.04 F here: weights of 0.05, hidden values about one) before the rounding
to bf16, which makes that one bf16 step (2^-7 of the value) more at most; an output adds as much of its largest row value."""
import pytest
import torch

from paper_2411_16786_amd import binding as B

import gpu_util as G
import plan_util as P

CASES = [
    # (T, T_max, d, F, E, k, n_shared, shares of the second GEMM when every pair is computed)
    (61, 70, 192, 3072, 4, 2, 0, 3),
    (40, 40, 1152, 3072, 8, 1, 0, 3),
    (90, 101, 1344, 3072, 5, 4, 0, 3),
    (30, 33, 576, 3072, 3, 2, 2, 3),          # two shared experts: four slots
    (30, 30, 576, 3072, 3, 3, 2, 3),          # five slots: more than the combine takes, the second pass adds
    (800, 800, 1152, 2048, 8, 2, 0, 2),
    (1200, 1201, 576, 2048, 9, 3, 0, 2),
]
ONLY_HERE = [
    # (T, T_max, d, F, E, k, n_shared, what the second GEMM is inside the layer call)
    (60, 61, 384, 1536, 16, 2, 0, "64x128/3"),
    (70, 70, 640, 2560, 4, 3, 1, "64x128/3"),
    (500, 500, 1152, 3072, 8, 2, 0, "128x128/2"),
]
HALF = [None, (B.REFRESH_ALL, 0), (B.REFRESH_ALG4, 0), (B.REFRESH_FRACTION_PAIR, 7)]


def test_the_second_gemm_is_split():
    for T, _, d, F, E, k, ns, shares in CASES:
        assert P.ffn_plans(T * (k + ns), E + ns, d, F)[1] == f"128x192deep/{shares}"


def test_split_inside_the_layer_call():
    for T, _, d, F, E, k, ns, shares in CASES:
        if k + ns <= 4:
            assert P.plan(False, d, F, T * (k + ns), E + ns, sums=True).endswith(f"/{shares}")
    for T, _, d, F, E, k, ns, tile in ONLY_HERE:
        assert P.plan(False, d, F, T * (k + ns), E + ns, sums=True) == tile
        assert "/" not in P.plan(False, d, F, T * (k + ns), E + ns)


@pytest.mark.parametrize("rows,E,d,F,tile", [
    (1024, 8, 768, 3072, "128x128/2"),           # three shares: nine tiles an XCD
    (1220, 4, 768, 3072, "128x128/2"),           # nine, with twelve slots a share: nine of 27 workgroups in one group of compute units
    (48, 8, 1280, 5120, "128x192deep/3"), (384, 8, 1280, 5120, "128x192deep/3"),
    (610, 8, 1024, 4096, "128x192deep/3"),
    (48, 8, 1152, 4608, "128x128/3"), (304, 8, 1152, 4608, "128x128/3"),      # nine, with eighteen slots
    (610, 8, 768, 3072, "128x128/3"),
])
def test_shares_run_in_one_round(rows, E, d, F, tile):
    assert P.plan(False, d, F, rows, E, sums=True) == tile


def separate_calls(ctx, buf, x, Wg, bg, w, policy, fuse, to_cache):
    T = x.shape[0]
    rows = T * ctx.slots if policy is None else ctx.moe_policy_refreshed_pairs(policy, T)[0]
    ctx.moe_gate(x, Wg, bg, buf.scores[:T], buf.expert_idx[:T])
    mask = None
    if policy is not None:
        mask = buf.mask[:T]
        ctx.moe_conditional_refresh(buf.scores[:T], buf.expert_idx[:T], policy, mask, buf.n_refresh, buf.workspace)
    ctx.moe_dispatch(x, buf.expert_idx[:T], mask, None if fuse else buf.x_packed, buf.counts, buf.offsets, buf.perm, buf.inv, buf.workspace)
    if to_cache:
        ctx.moe_expert_ffn_commit(x, buf.perm, buf.perm, buf.offsets, buf.seg_expert, rows, *w, None, mask, buf.H_cache, None, buf.workspace, T=T)
    elif fuse:
        ctx.moe_expert_ffn_rows(x, buf.perm, buf.offsets, buf.seg_expert, rows, *w, buf.h_packed, buf.workspace)
    else:
        ctx.moe_expert_ffn(buf.x_packed, buf.offsets, buf.seg_expert, rows, *w, buf.h_packed, buf.workspace)
    ctx.moe_combine(None if to_cache else buf.h_packed, buf.inv, buf.scores[:T], mask, buf.H_cache, buf.S_cache,
                    policy is not None and policy.use_fresh_scores, buf.y[:T])


def same_outputs(a, b, T, F, exact, what):
    """Outputs of the layer call (a) and of the separate calls (b): bit for bit, or, where only the layer call splits, within the bound above."""
    for name in ("y", "H_cache", "S_cache", "h_packed"):
        p, q = getattr(a, name), getattr(b, name)
        if exact or name == "S_cache":
            assert p is None or torch.equal(p, q), (name, what)
        elif p is not None:
            p, q = p.float(), q.float()
            scale = q.abs() if name != "y" else q.abs() + b.H_cache[:T].float().abs().amax() if b.H_cache is not None else q.abs() + b.h_packed.float().abs().amax()
            assert ((p - q).abs() <= 2.0 ** -7 * scale[:len(p)] + F / 16 * 2.0 ** -24 * 0.04 * F).all(), (name, what)
            assert (p == q).float().mean() > 0.9, (name, what)


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(CASES) + len(ONLY_HERE)))
@pytest.mark.parametrize("kind", range(len(HALF)))
def test_combine_adds_the_shares(case, kind):
    T, T_max, d, F, E, k, ns, _ = (CASES + ONLY_HERE)[case]
    if kind >= 2 and T > 100:
        pytest.skip("the refreshed rows of these sizes are not split")
    print(f"\nshares case {case} policy {kind}", flush=True)
    x, Wg, bg, *_ = G.small_inputs(91 + case, T, d, E, 64, "bf16")
    gen = torch.Generator(device=G.DEV).manual_seed(case)
    normal = lambda *s: torch.randn(s, generator=gen, device=G.DEV) * 0.05
    W1, W2 = normal(E + ns, F, d).bfloat16(), normal(E + ns, d, F).bfloat16()
    b1, b2 = (None, None) if case % 3 == 1 else (normal(E + ns, F), normal(E + ns, d))
    x, Wg, bg = G.to_dev(x, "bf16"), G.to_dev(Wg, "bf16"), G.f32_dev(bg)
    policy = None if HALF[kind] is None else B.Policy(HALF[kind][0], step_t=1, stride_n=2, n_units=T * k // 2 + HALF[kind][1],
                                                      use_fresh_scores=case % 2 == 1)
    for to_cache in ([False] if policy is None or ns else [True, False]):
        for fuse in [True] if to_cache else [True, False]:
            ctx = B.Context(T_max, d, F, E, k, "bf16", n_shared=ns)
            a, b = (B.LayerBuffers(ctx, G.DEV, with_cache=policy is not None) for _ in range(2))
            for buf in (a, b):
                buf.y.fill_(3.0)
                if policy is not None:
                    buf.H_cache.copy_(torch.linspace(-1, 1, buf.H_cache.numel(), device=G.DEV).view_as(buf.H_cache))
                    buf.S_cache.fill_(0.25)
            B.moe_layer_forward(ctx, a, x, Wg, bg, W1, b1, W2, b2, policy, fuse_gather=fuse, rows_to_cache=to_cache)
            separate_calls(ctx, b, x, Wg, bg, (W1, b1, W2, b2), policy, fuse, to_cache)
            torch.cuda.synchronize()
            same_outputs(a, b, T, F, case < len(CASES), (to_cache, fuse))
            assert a.x_packed is None or torch.equal(a.x_packed, b.x_packed), (to_cache, fuse)
            assert torch.isfinite(a.y[:T].float()).all() and a.y[:T].float().abs().sum() > 0


@pytest.mark.gpu
@pytest.mark.parametrize("case", [0, 1, 3, 5, 6])
@pytest.mark.parametrize("to_cache", [False, True])
def test_rows_beyond_the_bound_are_left_alone(case, to_cache):
    """A bound a few rows short: rows within it are computed as ever, those beyond it are neither read from the shares nor written, and the
    status call reports them."""
    T, T_max, d, F, E, k, ns, shares = CASES[case]
    if to_cache and ns:
        pytest.skip("rows_to_cache needs a shape without shared experts")
    short = T * (k + ns) - 5
    assert P.plan(False, d, F, short, E + ns, sums=True) == P.plan(False, d, F, short + 5, E + ns, sums=True)
    assert P.plan(False, d, F, short, E + ns, sums=True).endswith(f"/{shares}")
    print(f"\nbound short, case {case} to_cache={to_cache}", flush=True)
    x, Wg, bg, *_ = G.small_inputs(91 + case, T, d, E, 64, "bf16")
    gen = torch.Generator(device=G.DEV).manual_seed(case)
    normal = lambda *s: torch.randn(s, generator=gen, device=G.DEV) * 0.05
    w = (normal(E + ns, F, d).bfloat16(), normal(E + ns, F), normal(E + ns, d, F).bfloat16(), normal(E + ns, d))
    x, Wg, bg = G.to_dev(x, "bf16"), G.to_dev(Wg, "bf16"), G.f32_dev(bg)
    policy = B.Policy(B.REFRESH_ALL) if to_cache else None
    ctx = B.Context(T_max, d, F, E, k, "bf16", n_shared=ns)
    a, b = (B.LayerBuffers(ctx, G.DEV, with_cache=to_cache) for _ in range(2))
    for buf, rows in ((a, short + 5), (b, short)):
        buf.h_packed.fill_(0.5)
        if to_cache:
            buf.H_cache.fill_(0.5)
        B.moe_layer_forward(ctx, buf, x, Wg, bg, *w, policy, max_rows=rows)
    torch.cuda.synchronize()
    lost = a.perm[short:short + 5].long()                 # pairs of the rows beyond the bound
    p, q = (buf.H_cache.flatten(0, 1) if to_cache else buf.h_packed for buf in (a, b))
    rows = lost if to_cache else torch.arange(short, short + 5, device=G.DEV)
    assert (q[rows] == 0.5).all() and (p[rows] != 0.5).any()
    q[rows] = p[rows]
    assert torch.equal(p, q)
    whole = torch.ones(T, dtype=torch.bool, device=G.DEV)
    whole[lost // (k + ns)] = False                       # tokens of which no row is missing
    assert torch.equal(a.y[:T][whole], b.y[:T][whole]) and whole.any()
    ctx.moe_expert_ffn_status(a.workspace)
    with pytest.raises(B.MoeError):
        ctx.moe_expert_ffn_status(b.workspace)
