"""The layer in one native call: its argument struct as the header declares it, the same bits as the separate entry points in
every form (fused or materialised gather, rows scattered into the cache or not, shared experts), and what was refused."""
import os
import re

import pytest
import torch

from paper_2411_16786_amd import binding as B

import gpu_util as G


def test_layer_args_match_the_header():
    header = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "dice_moe.h")
    body = re.search(r"typedef struct moe_layer_args \{([^{}]*)\} moe_layer_args;", open(header).read(), re.S).group(1)
    declared = [(n, "*" in decl) for stmt in body.split(";") if stmt.strip()
                for decl in stmt.split(",") for n in re.findall(r"([A-Za-z_][A-Za-z0-9_]*)\s*$", decl)]
    bound = [(name, typ is B.ctypes.c_void_p) for name, typ in B.MoeLayerArgs._fields_]
    assert declared == bound


def layer_args(**over):
    """A call that passes every check, on dummy addresses: none of them is read on the paths below."""
    a = B.MoeLayerArgs(*([16] * 24), T=8, n_segments=4, max_rows=0, imply_rows=1, fuse_gather=1, rows_to_cache=0)
    for name, value in over.items():
        setattr(a, name, value)
    return a


POLICY = (B.REFRESH_ALG4, 1, 2, 0, 0)
REFUSED = [
    # (arguments that differ, policy, shared experts, status)
    ({"T": 65}, None, 0, B.MOE_ERR_SHAPE),
    ({"T": -1}, None, 0, B.MOE_ERR_SHAPE),
    ({"imply_rows": 0, "max_rows": -1}, None, 0, B.MOE_ERR_SHAPE),
    ({"imply_rows": 0, "max_rows": 129}, None, 0, B.MOE_ERR_SHAPE),
    ({"n_segments": 0}, None, 0, B.MOE_ERR_SHAPE),
    ({"n_segments": 1025}, None, 0, B.MOE_ERR_SHAPE),
    ({}, (B.REFRESH_ALG4, 1, 0, 0, 0), 0, B.MOE_ERR_POLICY),
    ({"imply_rows": 0, "max_rows": 8}, (99, 0, 1, 0, 0), 0, B.MOE_ERR_POLICY),
    ({"H_cache": None, "S_cache": None}, POLICY, 0, B.MOE_ERR_CACHE_COLD),
    ({"S_cache": None, "rows_to_cache": 1}, POLICY, 0, B.MOE_ERR_CACHE_COLD),
    ({"H_cache": None, "rows_to_cache": 1}, POLICY, 0, B.MOE_ERR_NULL),
    # the FFN writes rows into the cache only with a policy, the fused gather and no shared experts
    ({"rows_to_cache": 1}, None, 0, B.MOE_ERR_NULL),
    ({"rows_to_cache": 1, "fuse_gather": 0}, POLICY, 0, B.MOE_ERR_NULL),
    ({"rows_to_cache": 1}, POLICY, 2, B.MOE_ERR_NULL),
    ({"workspace": None}, None, 0, B.MOE_ERR_WORKSPACE),
    ({"h_packed": None}, None, 0, B.MOE_ERR_NULL),
    ({"h_packed": None}, POLICY, 0, B.MOE_ERR_NULL),
    ({"x_packed": None, "fuse_gather": 0}, None, 0, B.MOE_ERR_NULL),
    ({"mask": None}, POLICY, 0, B.MOE_ERR_NULL),
    ({"n_refresh": None}, POLICY, 0, B.MOE_ERR_NULL),
] + [({name: None}, None, 0, B.MOE_ERR_NULL) for name in ("x", "Wg", "W1", "W2", "scores", "expert_idx", "counts", "offsets", "perm",
                                                          "inv", "seg_expert", "y")]


@pytest.mark.parametrize("case", range(len(REFUSED)))
def test_refused_before_the_first_launch(case):
    """Host-visible errors of any part come back before the first part is launched (without a GPU, a launch would be MOE_ERR_HIP)."""
    over, policy, n_shared, status = REFUSED[case]
    ctx = B.Context(T_max=64, d=64, F=256, E=4, k=2, dtype="f32", n_shared=n_shared)
    pol = None if policy is None else B.ctypes.byref(B.MoePolicy(*policy))
    assert B.lib().moe_layer_forward(ctx._h, B.ctypes.byref(layer_args(**over)), pol, None) == status
    assert B.lib().moe_last_error(ctx._h) != b""


FORMS = [
    # (policy, n_shared, keywords)
    (None, 0, {}),
    (None, 2, {"fuse_gather": False}),
    (B.Policy(B.REFRESH_ALG4, step_t=1, stride_n=2), 0, {}),
    (B.Policy(B.REFRESH_ALG4, step_t=1, stride_n=2), 0, {"rows_to_cache": False}),
    (B.Policy(B.REFRESH_FRACTION_TOKEN, n_units=20, use_fresh_scores=True), 1, {}),
    (B.Policy(B.REFRESH_FRACTION_PAIR, n_units=75), 0, {"fuse_gather": False, "max_rows": 90}),
]


@pytest.mark.gpu
@pytest.mark.parametrize("form", range(len(FORMS)))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_one_call_equals_the_separate_ones(form, dtype):
    policy, ns, kw = FORMS[form]
    T, T_max, d, F, E, k = 61, 70, 64, 192, 5, 2
    x, Wg, bg, *_ = G.small_inputs(81, T, d, E, F, dtype)
    *_, W1, b1, W2, b2 = G.small_inputs(82, T, d, E + ns, F, dtype)
    ctx = B.Context(T_max, d, F, E, k, dtype, n_shared=ns)
    dev = [G.to_dev(x, dtype), G.to_dev(Wg, dtype), G.f32_dev(bg), G.to_dev(W1, dtype), G.f32_dev(b1), G.to_dev(W2, dtype), G.f32_dev(b2)]
    a, b = (B.LayerBuffers(ctx, G.DEV, with_cache=policy is not None) for _ in range(2))
    for buf in (a, b):
        buf.y.fill_(3.0)
        if policy is not None:
            buf.H_cache.copy_(torch.linspace(-1, 1, buf.H_cache.numel(), device=G.DEV).view_as(buf.H_cache))
            buf.S_cache.fill_(0.25)
    B.moe_layer_forward(ctx, a, *dev, policy, **kw)

    fuse = kw.get("fuse_gather", True)
    to_cache = kw.get("rows_to_cache", policy is not None and fuse and ns == 0)
    rows = kw.get("max_rows", T * ctx.slots if policy is None else ctx.moe_policy_refreshed_pairs(policy, T)[0])
    xd, Wgd, bgd, *w = dev
    ctx.moe_gate(xd, Wgd, bgd, b.scores[:T], b.expert_idx[:T])
    mask = None
    if policy is not None:
        mask = b.mask[:T]
        ctx.moe_conditional_refresh(b.scores[:T], b.expert_idx[:T], policy, mask, b.n_refresh, b.workspace)
    ctx.moe_dispatch(xd, b.expert_idx[:T], mask, None if fuse else b.x_packed, b.counts, b.offsets, b.perm, b.inv, b.workspace)
    if to_cache:
        ctx.moe_expert_ffn_commit(xd, b.perm, b.perm, b.offsets, b.seg_expert, rows, *w, None, mask, b.H_cache, None, b.workspace, T=T)
    elif fuse:
        ctx.moe_expert_ffn_rows(xd, b.perm, b.offsets, b.seg_expert, rows, *w, b.h_packed, b.workspace)
    else:
        ctx.moe_expert_ffn(b.x_packed, b.offsets, b.seg_expert, rows, *w, b.h_packed, b.workspace)
    ctx.moe_combine(None if to_cache else b.h_packed, b.inv, b.scores[:T], mask, b.H_cache, b.S_cache,
                    policy is not None and policy.use_fresh_scores, b.y[:T])
    torch.cuda.synchronize()
    for name in ("y", "H_cache", "S_cache", "h_packed", "x_packed"):
        p, q = getattr(a, name), getattr(b, name)
        assert p is None or torch.equal(p, q), name
    for name in ("scores", "expert_idx", "perm", "inv"):
        n = T if name in ("scores", "expert_idx") else T * ctx.slots
        assert torch.equal(getattr(a, name)[:n], getattr(b, name)[:n]), name
    assert (G.to_np(a.y)[T:] == 3.0).all()


@pytest.mark.gpu
def test_one_call_refuses_what_the_separate_ones_refuse():
    T, d, F, E, k = 16, 64, 64, 4, 2
    x, Wg, bg, W1, b1, W2, b2 = G.small_inputs(83, T, d, E, F, "f32")
    ctx = B.Context(T, d, F, E, k, "f32")
    dev = [G.to_dev(x, "f32"), G.to_dev(Wg, "f32"), G.f32_dev(bg), G.to_dev(W1, "f32"), G.f32_dev(b1), G.to_dev(W2, "f32"), G.f32_dev(b2)]
    buf = B.LayerBuffers(ctx, G.DEV)

    def status(**kw):
        with pytest.raises(B.MoeError) as err:
            B.moe_layer_forward(ctx, buf, *kw.pop("dev", dev), **kw)
        return err.value.status

    assert status(max_rows=-1) == B.MOE_ERR_SHAPE
    assert status(max_rows=T * k + 1) == B.MOE_ERR_SHAPE
    assert status(dev=[torch.cat([dev[0], dev[0]])] + dev[1:]) == B.MOE_ERR_SHAPE                # T beyond T_max
    assert status(policy=B.Policy(77)) == B.MOE_ERR_POLICY
    assert status(policy=B.Policy(B.REFRESH_ALL), rows_to_cache=False) == B.MOE_ERR_CACHE_COLD   # no caches in buf
    with pytest.raises(ValueError):
        B.moe_layer_forward(ctx, buf, *dev, rows_to_cache=True)
    with pytest.raises(ValueError):
        B.moe_layer_forward(ctx, buf, dev[0].t(), *dev[1:])
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("n_shared,over,status", [(2, {}, B.MOE_ERR_NULL), (0, {"imply_rows": 0, "max_rows": -1}, B.MOE_ERR_SHAPE),
                                                  (0, {"S_cache": None}, B.MOE_ERR_CACHE_COLD)])
def test_a_refused_call_writes_nothing(n_shared, over, status):
    T, d, F, E, k = 16, 64, 64, 4, 2
    x, Wg, bg, *_ = G.small_inputs(84, T, d, E, F, "f32")
    *_, W1, b1, W2, b2 = G.small_inputs(85, T, d, E + n_shared, F, "f32")
    ctx = B.Context(T, d, F, E, k, "f32", n_shared=n_shared)
    dev = {"x": G.to_dev(x, "f32"), "Wg": G.to_dev(Wg, "f32"), "W1": G.to_dev(W1, "f32"), "W2": G.to_dev(W2, "f32")}
    buf = B.LayerBuffers(ctx, G.DEV, with_cache=True)
    dev |= {n: getattr(buf, n) for n in ("scores", "expert_idx", "mask", "n_refresh", "h_packed", "counts", "offsets", "perm", "inv",
                                         "seg_expert", "H_cache", "S_cache", "y", "workspace")}
    outputs = ("scores", "expert_idx", "mask", "n_refresh", "h_packed", "counts", "offsets", "perm", "inv", "H_cache", "S_cache", "y")
    for name in outputs:
        dev[name].fill_(7)
    a = B.MoeLayerArgs(**{n: t.data_ptr() for n, t in dev.items()}, T=T, n_segments=ctx.experts, imply_rows=1, fuse_gather=1, rows_to_cache=1)
    for name, value in over.items():
        setattr(a, name, value)
    pol = B.MoePolicy(*POLICY)
    assert B.lib().moe_layer_forward(ctx._h, B.ctypes.byref(a), B.ctypes.byref(pol), None) == status
    torch.cuda.synchronize()
    for name in outputs:
        assert (dev[name] == 7).all(), name
