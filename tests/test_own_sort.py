"""Layers of up to 1024 pairs, whose first GEMM sorts the pairs itself: every buffer the layer leaves behind has the bits of the separate
calls (with a dispatch of their own), at the pair counts where the sort takes another number of steps, on every kernel that does it, with every
elementwise policy, shared experts, empty experts, and a bound on the rows that the host gives."""
import pytest
import torch

from paper_2411_16786_amd import binding as B

import gpu_util as G
import plan_util as P
from test_layer_sums import separate_calls

KERNELS = [
    # (dtype, d, F, E): first GEMM on
    ("bf16", 384, 512, 16),       # 64 x 128 tiles
    ("bf16", 1152, 1472, 16),     # 128 x 192, three stages, eight wavefronts
    ("f32", 256, 192, 5),         # direct, two stages of the ring
    ("f32", 64, 80, 64),          # direct
    ("f32", 384, 192, 5),         # ring
]
POLICIES = [None, (B.REFRESH_ALL, 0), (B.REFRESH_ALG4, 1), (B.REFRESH_ALG4_HIGH, 1), (B.REFRESH_ALG4_RANDOM, 1), (B.REFRESH_NONE, 0)]
SIZES = [(1, 1, 0), (32, 2, 0), (33, 2, 0), (85, 2, 1), (171, 3, 0), (512, 2, 0), (341, 3, 0), (513, 2, 0)]


def test_the_kernels_are_those():
    assert P.plan(True, 512, 384, 1024, 16) == "64x128" and P.plan(True, 512, 384, 64, 16) == "64x128"
    assert P.plan(True, 1472, 1152, 1024, 16) == "128x192deep" and P.plan(True, 1472, 1152, 64, 16) == "128x192deep"
    for rows in (2, 1024):
        assert [P.f32_plans(rows, E, d, F)[0] for dtype, d, F, E in KERNELS if dtype == "f32"] == ["direct32", "direct32", "ring32"]


def refreshed(kind, T, k, ns):
    return {None: T * k, B.REFRESH_ALL: T * k, B.REFRESH_NONE: 0}.get(kind, T) + T * ns


@pytest.mark.parametrize("kernel", range(len(KERNELS)))
@pytest.mark.parametrize("size", SIZES)
def test_they_sort_the_pairs(kernel, size):
    """... up to 1024 pairs, if any is refreshed."""
    dtype, d, F, E = KERNELS[kernel]
    T, k, ns = size
    for entry in POLICIES:
        rows = refreshed(entry and entry[0], T, k, ns)
        assert P.sorts_pairs(dtype, T, k + ns, E + ns, d, F, rows) == (T * (k + ns) <= 1024 and rows > 0), entry


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", range(len(KERNELS)))
@pytest.mark.parametrize("size", SIZES)
def test_own_sort(kernel, size):
    dtype, d, F, E = KERNELS[kernel]
    T, k, ns = size
    print(f"\nown sort {KERNELS[kernel]} {size}", flush=True)
    x, Wg, bg, *_ = G.small_inputs(41, T, d, E, 64, dtype)
    bg[E // 2] = -30.0                                   # an expert without rows
    gen = torch.Generator(device=G.DEV).manual_seed(5)
    normal = lambda *s: torch.randn(s, generator=gen, device=G.DEV) * 0.05
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    w = (normal(E + ns, F, d).to(dt), normal(E + ns, F), normal(E + ns, d, F).to(dt), normal(E + ns, d)) if E + ns <= 64 else None
    if w is None:
        pytest.skip("64 experts at most")
    x, Wg, bg = G.to_dev(x, dtype), G.to_dev(Wg, dtype), G.f32_dev(bg)
    for entry in POLICIES:
        policy = None if entry is None else B.Policy(entry[0], step_t=entry[1], stride_n=2, n_units=77)
        ctx = B.Context(T + 2, d, F, E, k, dtype, n_shared=ns)
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
        for name in ("scores", "expert_idx", "mask", "n_refresh", "counts", "offsets", "perm", "inv", "y", "h_packed", "H_cache", "S_cache"):
            p, q = getattr(a, name), getattr(b, name)
            assert p is None or torch.equal(p, q), (entry, name)
        ctx.moe_expert_ffn_status(a.workspace)


@pytest.mark.gpu
def test_rows_beyond_the_bound_are_reported():
    T, d, F, E, k = 64, 384, 512, 16, 2
    x, Wg, bg, W1, b1, W2, b2 = G.small_inputs(43, T, d, E, F, "bf16")
    ctx = B.Context(T, d, F, E, k, "bf16")
    buf = B.LayerBuffers(ctx, G.DEV)
    dev = [G.to_dev(x, "bf16"), G.to_dev(Wg, "bf16"), G.f32_dev(bg), G.to_dev(W1, "bf16"), G.f32_dev(b1), G.to_dev(W2, "bf16"), G.f32_dev(b2)]
    B.moe_layer_forward(ctx, buf, *dev, max_rows=T * k)
    ctx.moe_expert_ffn_status(buf.workspace)
    B.moe_layer_forward(ctx, buf, *dev, max_rows=T * k - 1)
    with pytest.raises(B.MoeError):
        ctx.moe_expert_ffn_status(buf.workspace)
