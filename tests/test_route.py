"""Router, refresh decision and dispatch in one call: the same bits as the three separate calls, for every policy, at the pair counts where the
dispatch takes another form (256, 1024, 2048, 4096), with shared experts, equal scores, and nothing or everything selected."""
import pytest
import torch

from paper_2411_16786_amd import binding as B

import gpu_util as G

POLICIES = [
    # (kind, step_t, units of n_units: "T" tokens, "N" routed pairs)
    (None, 0, 0, ""),
    (B.REFRESH_ALL, 0, 0, ""), (B.REFRESH_NONE, 0, 0, ""),
    (B.REFRESH_ALG4, 1, 0, ""), (B.REFRESH_ALG4, 2, 0, ""), (B.REFRESH_ALG4_HIGH, 1, 0, ""), (B.REFRESH_ALG4_RANDOM, 3, 12345, ""),
    (B.REFRESH_FRACTION_TOKEN, 0, 0.0, "T"), (B.REFRESH_FRACTION_TOKEN, 0, 0.37, "T"), (B.REFRESH_FRACTION_TOKEN, 0, 1.0, "T"),
    (B.REFRESH_FRACTION_PAIR, 0, 0.3, "N"), (B.REFRESH_FRACTION_PAIR, 0, 0.8, "N"), (B.REFRESH_FRACTION_PAIR, 0, 1.0, "N"),
]
SIZES = [
    # (T, E, k, n_shared)
    (1, 4, 2, 0),
    (128, 4, 2, 0), (129, 5, 2, 0), (85, 4, 1, 2),
    (256, 8, 1, 0), (1024, 8, 1, 0), (1025, 8, 1, 0), (683, 16, 2, 1),
    (4096, 8, 1, 0), (2048, 64, 2, 0), (2049, 8, 2, 0), (5000, 8, 3, 0),
    (17000, 4, 1, 0),
]


def policy_of(entry, T, k):
    kind, step, units, of = entry
    if kind is None:
        return None
    n = int(units * (T if of == "T" else T * k)) if of else units
    return B.Policy(kind, step_t=step, stride_n=2, n_units=n)


@pytest.mark.gpu
@pytest.mark.parametrize("size", SIZES)
def test_route_equals_the_separate_calls(size):
    T, E, k, ns = size
    print(f"\nroute {size}", flush=True)
    x, Wg, bg, *_ = G.small_inputs(61, T, 64, E, 64, "bf16")
    if T > 4:
        x[T // 2:T // 2 + T // 4] = x[0]          # equal rows: equal scores across the cut
    x, Wg, bg = G.to_dev(x, "bf16"), G.to_dev(Wg, "bf16"), G.f32_dev(bg)
    for entry in POLICIES:
        policy = policy_of(entry, T, k)
        for packed in (False, True):
            ctx = B.Context(T + 3, 64, 64, E, k, "bf16", n_shared=ns)
            a, b = (B.LayerBuffers(ctx, G.DEV, with_debug=True) for _ in range(2))
            for buf in (a, b):
                for t in (buf.scores, buf.expert_idx, buf.mask, buf.n_refresh, buf.counts, buf.offsets, buf.perm, buf.inv, buf.x_packed):
                    t.fill_(7)
            ctx.moe_route(x, Wg, bg, policy, a.scores, a.expert_idx, a.mask, a.n_refresh, a.x_packed if packed else None, a.counts,
                          a.offsets, a.perm, a.inv, a.workspace, a.probs, a.logits)
            ctx.moe_gate(x, Wg, bg, b.scores, b.expert_idx, b.probs, b.logits)
            if policy is not None:
                ctx.moe_conditional_refresh(b.scores[:T], b.expert_idx[:T], policy, b.mask[:T], b.n_refresh, b.workspace)
            ctx.moe_dispatch(x, b.expert_idx[:T], None if policy is None else b.mask[:T], b.x_packed if packed else None, b.counts, b.offsets,
                             b.perm, b.inv, b.workspace)
            torch.cuda.synchronize()
            for name in ("scores", "expert_idx", "mask", "n_refresh", "counts", "offsets", "perm", "inv", "x_packed"):
                assert torch.equal(getattr(a, name), getattr(b, name)), (entry, packed, name)


def test_route_refuses_before_the_first_launch():
    ctx = B.Context(T_max=64, d=64, F=256, E=4, k=2, dtype="f32")
    call = lambda policy=None, **over: B.lib().moe_route(ctx._h, *[over.get(n, 16) for n in ("x", "Wg", "bg")], over.get("T", 8),
                                                         None if policy is None else B.ctypes.byref(B.MoePolicy(*policy)),
                                                         *[over.get(n, 16) for n in ("scores", "expert_idx", "probs", "logits", "mask", "n_refresh",
                                                                                     "x_packed", "counts", "offsets", "perm", "inv", "workspace")], None)
    assert call(T=65) == B.MOE_ERR_SHAPE
    assert call(policy=(99, 0, 1, 0, 0)) == B.MOE_ERR_POLICY
    assert call(policy=(B.REFRESH_ALL, 0, 1, 0, 0), mask=None) == B.MOE_ERR_NULL
    for name in ("x", "Wg", "scores", "expert_idx", "counts", "offsets", "perm", "inv"):
        assert call(**{name: None}) == B.MOE_ERR_NULL
