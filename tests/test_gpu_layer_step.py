"""The whole step as one call against the calls of the single steps: the same outputs, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2506_07366_amd import workloads as wl
from paper_2506_07366_amd.layer import MoELayer, to_device

pytestmark = pytest.mark.gpu


def outputs(layer):
    p = layer.perm
    names = ("topk_idx", "topk_w", "hist", "slot_expert", "slot_quota", "rank_load_pred", "n_iters", "out")
    res = {n: getattr(layer, n).clone() for n in names}
    res.update({n: p[n].clone() for n in ("seg_offsets", "row_of_assign", "assign_of_row", "rank_load")})
    return res


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("T,E,k,G,S,dtype", [
    (1, 8, 2, 8, 2, "bf16"),          # one token
    (7, 2, 1, 2, 1, "f32"),           # two lanes per token, no spare slot
    (33, 3, 2, 2, 3, "bf16"),         # four lanes, an uneven home placement
    (256, 8, 2, 8, 3, "f32"),
    (1024, 16, 2, 4, 5, "bf16"),      # 2048 assignments: the last in one workgroup with predicted ids
    (1025, 16, 2, 4, 5, "bf16"),
    (512, 24, 6, 12, 3, "bf16"),      # 3072: the last in one workgroup without
    (513, 24, 6, 12, 3, "bf16"),
    (2048, 64, 8, 16, 5, "bf16"),     # 16384: the last whose predicted ids one workgroup counts
    (2049, 64, 8, 16, 5, "bf16"),
    (100, 256, 4, 32, 10, "bf16"),    # the planner's launch is shared up to here
    (100, 257, 4, 32, 10, "bf16"),
    (100, 32, 4, 33, 2, "bf16"),
    (100, 22, 4, 2, 11, "bf16"),
    (300, 600, 8, 64, 16, "bf16"),    # tables too large for one workgroup
])
def test_step_equals_single_calls(T, E, k, G, S, dtype, mode):
    d, ffn = 64, 64
    cfg = wl.MoEConfig("st", T=T, d=d, ffn=ffn, E=E, k=k, G=G, S=S, dtype=dtype, mode=mode, seed=61)
    rng = np.random.default_rng([62, T, E, mode])
    logits = torch.from_numpy(rng.standard_normal((T, E)).astype(np.float32) - np.log1p(np.arange(E))[None]
                              .astype(np.float32)).cuda()
    x = to_device(wl.to_storage(rng.standard_normal((T, d)).astype(np.float32), dtype), dtype)
    ws = [to_device(wl.to_storage((rng.standard_normal(s) * 0.02).astype(np.float32), dtype), dtype)
          for s in ((E, d, ffn), (E, d, ffn), (E, ffn, d))]
    pred_idx = torch.topk(logits + 0.5 * torch.randn_like(logits), k, dim=1).indices.to(torch.int32).contiguous()
    hist_pred = torch.bincount(pred_idx.reshape(-1).long(), minlength=E).to(torch.int32)
    for gather, weights, act in ((False, False, "swiglu"), (True, False, "swiglu"), (True, True, "swiglu"),
                                 (False, False, "relu")):
        layer = MoELayer(cfg.replace(act=act), fused_gather=gather, fused_weights=weights)
        layer.set_weights(*ws)
        layer.route(logits)
        layer.histogram()
        layer.plan(mode, hist_pred, pred_idx)
        layer.permute(mode, x, pred_idx)
        layer.ffn()
        layer.combine()
        want = outputs(layer)
        plan_hist = layer.hist_plan.clone()
        for t in (*(layer.perm[n] if n in layer.perm else getattr(layer, n) for n in want), layer.hist_plan, layer.y_perm,
                  *(v for v in (layer.perm["x_perm"],) if v is not None)):
            t.fill_(-7)
        assert layer._one_call(logits, x, hist_pred, pred_idx, mode)
        got = outputs(layer)
        for n, v in want.items():
            assert torch.equal(got[n], v), n
        if mode == 2:
            assert torch.equal(layer.hist_plan, plan_hist)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("T,E,k,G,S", [
    (64, 16, 2, 4, 5),        # one workgroup permutes, routing and plan would share a launch
    (3000, 16, 8, 4, 5),      # 24000 ids: three launches permute, a launch of its own counts the predicted ids
    (100, 300, 4, 32, 10),    # routing and plan never share a launch
])
def test_step_on_its_own_outputs_as_prediction(T, E, k, G, S, mode):
    """A perfect prediction is the step's own topk_idx (or hist): the step uses what it has just written there,
    as the single calls do, and not what an earlier batch left."""
    cfg = wl.MoEConfig("own", T=T, d=64, ffn=64, E=E, k=k, G=G, S=S, dtype="bf16", mode=mode, seed=63)
    gen = torch.Generator(device="cuda").manual_seed(64)
    ws = [torch.randn(s, device="cuda", generator=gen).mul_(0.02).to(torch.bfloat16)
          for s in ((E, 64, 64), (E, 64, 64), (E, 64, 64))]
    want_layer, layer = MoELayer(cfg), MoELayer(cfg)
    want_layer.set_weights(*ws)
    layer.set_weights(*ws)
    skew = torch.log1p(torch.arange(E, device="cuda", dtype=torch.float32))
    for batch in range(2):                             # (the second finds the first one's ids and counts in place)
        logits = torch.randn((T, E), device="cuda", generator=gen) + (skew if batch else -skew)
        x = torch.randn((T, 64), device="cuda", generator=gen).to(torch.bfloat16)
        want_layer.route(logits)
        want_layer.histogram()
        want_layer.plan(mode, want_layer.hist, want_layer.topk_idx)
        want_layer.permute(mode, x, want_layer.topk_idx)
        want_layer.ffn()
        want_layer.combine()
        if batch == 0:
            layer.hist.zero_()
            layer.topk_idx.zero_()
        assert layer._one_call(logits, x, layer.hist, layer.topk_idx, mode)
        want, got = outputs(want_layer), outputs(layer)
        for n, v in want.items():
            assert torch.equal(got[n], v), n


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("T,E,k,G,S", [(64, 16, 2, 4, 5),      # one workgroup permutes
                                       (700, 12, 4, 5, 3),     # the same without predicted ids, an uneven home placement
                                       (3000, 16, 8, 4, 5)])
def test_step_with_ids_of_no_expert(T, E, k, G, S, mode):
    """A row of NaN logits gets ids outside [0, E): no histogram counts them, whoever makes it, and what follows
    from the counts is the same."""
    cfg = wl.MoEConfig("nan", T=T, d=64, ffn=64, E=E, k=k, G=G, S=S, dtype="bf16", mode=mode, seed=65)
    gen = torch.Generator(device="cuda").manual_seed(66)
    layer = MoELayer(cfg)
    layer.set_weights(*[torch.randn((E, 64, 64), device="cuda", generator=gen).mul_(0.02).to(torch.bfloat16)
                        for _ in range(3)])
    logits = torch.randn((T, E), device="cuda", generator=gen)
    logits[[0, T // 2, T - 1]] = float("nan")
    x = torch.randn((T, 64), device="cuda", generator=gen).to(torch.bfloat16)
    pred_idx = torch.randint(0, E, (T, k), device="cuda", generator=gen, dtype=torch.int32)
    pred_idx[1], pred_idx[2] = -1, E
    hist_pred = torch.bincount(pred_idx[3:].reshape(-1).long(), minlength=E).to(torch.int32)
    layer.route(logits)
    layer.histogram()
    layer.plan(mode, hist_pred, pred_idx)
    layer.permute(mode, x, pred_idx)
    layer.ffn()
    layer.combine()
    want = outputs(layer)
    assert int(want["hist"].sum()) == (T - 3) * k
    for n in want:
        (layer.perm[n] if n in layer.perm else getattr(layer, n)).fill_(-7)
    assert layer._one_call(logits, x, hist_pred, pred_idx, mode)
    got = outputs(layer)
    for n, v in want.items():
        assert torch.equal(got[n].nan_to_num(3.5), v.nan_to_num(3.5)), n


def test_step_leaves_other_inputs_to_the_single_calls():
    """Inputs that are not the layer's own sizes keep the behaviour (and the errors) of the single calls."""
    cfg = wl.CONFIGS["mid_bf16"]
    layer = MoELayer(cfg)
    x = torch.zeros((cfg.T, cfg.d), dtype=torch.bfloat16, device="cuda")
    logits = torch.zeros((cfg.T, cfg.E), device="cuda")
    hist = torch.ones(cfg.E, dtype=torch.int32, device="cuda")
    assert not layer._one_call(logits, x, hist, None, 1)              # no weights yet
    with pytest.raises(Exception):
        layer.step(logits, x, hist_pred=hist)
    layer.packed = torch.empty(256, dtype=torch.uint8, device="cuda")  # (never read below)
    assert not layer._one_call(logits, x, None, None, 1)
    assert not layer._one_call(logits, x, hist, None, 2)
    assert not layer._one_call(logits[:-1], x, hist, None, 1)
    assert not layer._one_call(logits, x.float(), hist, None, 1)
    assert not layer._one_call(logits, x, hist, None, 3)
    with pytest.raises(Exception):
        layer.step(logits.double(), x, hist_pred=hist)
    with pytest.raises(Exception):
        layer.step(logits, x, hist_pred=hist.long())


@pytest.mark.parametrize("T,d,E,k,dtype,act,stream", [
    (1, 64, 8, 2, "bf16", "swiglu", -1),        # one token: fewer wavefronts than a workgroup has
    (37, 2048, 8, 2, "bf16", "swiglu", 1),      # weights streamed, first form; rows shared by several wavefronts
    (37, 2112, 8, 16 // 2, "bf16", "relu", 2),  # second form, a row that is no whole number of pieces per lane
    (200, 4096, 16, 4, "bf16", "swiglu", 0),    # tiles
    (5003, 192, 4, 1, "bf16", "relu", 0),       # short rows, several per wavefront, the last wavefront with fewer
    (777, 1088, 8, 3, "bf16", "swiglu", -1),
    (1, 4, 3, 1, "f32", "swiglu", -1),          # one piece a row
    (515, 132, 8, 2, "f32", "relu", -1),
])
def test_step_copies_every_row(T, d, E, k, dtype, act, stream):
    """x_perm of a whole step, copied beside the first product: every row, nothing behind the last one."""
    from paper_2506_07366_amd import binding as B
    cfg = wl.MoEConfig("copy", T=T, d=d, ffn=64, E=E, k=k, G=2, S=E, dtype=dtype, mode=0, seed=67, act=act)
    gen = torch.Generator(device="cuda").manual_seed(68)
    layer = MoELayer(cfg)
    dt = layer.out.dtype
    layer.set_weights(*[torch.randn(s, device="cuda", generator=gen).mul_(0.02).to(dt)
                        for s in ((E, d, 64), (E, d, 64), (E, 64, d))])
    store = torch.full((cfg.A + 8, d), -7, dtype=dt, device="cuda")
    layer.perm["x_perm"] = store[:cfg.A]
    logits = torch.randn((T, E), device="cuda", generator=gen)
    x = torch.randn((T, d), device="cuda", generator=gen).to(dt)
    B.moe_grouped_ffn_set_option(B.FFN_OPT_STREAM, stream)
    try:
        assert layer._one_call(logits, x, None, None, 0)
    finally:
        B.moe_grouped_ffn_set_option(B.FFN_OPT_STREAM, -1)
    assert torch.equal(store[:cfg.A], x[layer.perm["assign_of_row"].long() // k])
    assert bool((store[cfg.A:] == -7).all())


@pytest.mark.parametrize("gather", [False, True])
@pytest.mark.parametrize("T", [200, 3000])           # one workgroup permutes, several
def test_step_with_scratch_shared_by_its_stages(T, gather):
    """The permutation's scratch is the FFN's, or lies in x_perm: nothing of the one is wanted once the other is written."""
    cfg = wl.MoEConfig("shared", T=T, d=128, ffn=128, E=16, k=4, G=4, S=5, dtype="bf16", mode=1, seed=69)
    gen = torch.Generator(device="cuda").manual_seed(70)
    ws = [torch.randn(s, device="cuda", generator=gen).mul_(0.02).to(torch.bfloat16)
          for s in ((16, 128, 128), (16, 128, 128), (16, 128, 128))]
    logits = torch.randn((T, 16), device="cuda", generator=gen)
    x = torch.randn((T, 128), device="cuda", generator=gen).to(torch.bfloat16)
    hist = torch.bincount(torch.topk(logits, 4, dim=1).indices.reshape(-1), minlength=16).to(torch.int32)
    got = []
    for shared in (None, "ffn", "x_perm"):
        layer = MoELayer(cfg, fused_gather=gather)
        layer.set_weights(*ws)
        if shared == "ffn":
            layer.ws_perm = layer.ws_ffn = torch.empty(max(layer.ws_perm.numel(), layer.ws_ffn.numel()), dtype=torch.uint8,
                                                       device="cuda")
        elif shared == "x_perm" and not gather:
            layer.ws_perm = layer.perm["x_perm"].view(torch.uint8).reshape(-1)
        assert layer._one_call(logits, x, hist, None, 1)
        got.append(outputs(layer))
    for other in got[1:]:
        for n, v in got[0].items():
            assert torch.equal(other[n], v), n


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("T,E,k,G,S", [
    (3073, 8, 1, 4, 3),        # just past one workgroup: 13 chunks, the last of one token
    (1638, 256, 5, 32, 10),    # chunks of 51 tokens, 33 of them; the most experts that share the planner's launch
    (16384, 24, 2, 12, 3),     # 128 chunks of 256 assignments
    (16400, 24, 2, 12, 3),     # chunks of 512
    (70001, 3, 3, 2, 3),       # chunks of 2046 with an odd last one
])
def test_step_permuted_by_many_workgroups(T, E, k, G, S, mode):
    """Histogram and plan that the permuting launches make, at either side of their chunks' sizes."""
    test_step_equals_single_calls(T, E, k, G, S, "bf16", mode)


@pytest.mark.parametrize("gather", [False, True])
@pytest.mark.parametrize("T", [300, 3000])           # one workgroup permutes and streams; several, both products in one launch
def test_step_with_buffers_that_share_memory(T, gather):
    """y_perm on x or on x_perm, x in the FFN's scratch (with a copy of its rows), the two histograms of the Token-to-Expert
    plan in one place: the step reads what is read late before it writes there."""
    E, k, d, ffn = 8, 2, 1024, 2048
    cfg = wl.MoEConfig("alias", T=T, d=d, ffn=ffn, E=E, k=k, G=4, S=3, dtype="bf16", mode=2, seed=71)
    gen = torch.Generator(device="cuda").manual_seed(72)
    ws = [torch.randn(s, device="cuda", generator=gen).mul_(0.02).to(torch.bfloat16)
          for s in ((E, d, ffn), (E, d, ffn), (E, ffn, d))]
    logits = torch.randn((T, E), device="cuda", generator=gen)
    x = torch.randn((T, d), device="cuda", generator=gen).to(torch.bfloat16)
    pred_idx = torch.topk(logits, k, dim=1).indices.to(torch.int32).contiguous()
    res = {}
    for how in ("none", "y on x", "y on x_perm", "x in scratch", "one histogram"):
        if gather and how in ("y on x_perm", "x in scratch"):
            continue
        layer = MoELayer(cfg, fused_gather=gather)
        layer.set_weights(*ws)
        given = x.clone()
        if how == "y on x":
            layer.y_perm[:T].copy_(x)
            given = layer.y_perm[:T]
        elif how == "y on x_perm":
            layer.y_perm = layer.perm["x_perm"]
        elif how == "x in scratch":
            given = layer.ws_ffn[:T * d * 2].view(torch.bfloat16).reshape(T, d)
            given.copy_(x)
        elif how == "one histogram":
            layer.hist_plan = layer.hist
        assert layer._one_call(logits, given, None, pred_idx, 2)
        res[how] = outputs(layer)
        if not gather and how != "y on x_perm":
            assert torch.equal(layer.perm["x_perm"], x[layer.perm["assign_of_row"].long() // k]), how
    for how, got in res.items():
        for n, v in res["none"].items():
            if how == "x in scratch" and n == "out":   # (rows in place: the same sums)
                assert torch.allclose(got[n].float(), v.float(), rtol=1e-2, atol=1e-3), n
            else:
                assert torch.equal(got[n], v), (how, n)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("T", [300, 3000, 20000])
def test_step_with_outputs_in_the_logits(T, mode):
    """Histogram and plan on logits that are of no further use, at their start (read by the first workgroup) and their end."""
    E, k, d = 16, 2, 64
    cfg = wl.MoEConfig("inlog", T=T, d=d, ffn=64, E=E, k=k, G=4, S=5, dtype="bf16", mode=mode, seed=73)
    gen = torch.Generator(device="cuda").manual_seed(74)
    ws = [torch.randn(s, device="cuda", generator=gen).mul_(0.02).to(torch.bfloat16) for s in ((E, d, 64), (E, d, 64), (E, 64, d))]
    logits = torch.randn((T, E), device="cuda", generator=gen)
    x = torch.randn((T, d), device="cuda", generator=gen).to(torch.bfloat16)
    pred_idx = torch.topk(logits + 0.5 * torch.randn((T, E), device="cuda", generator=gen), k, dim=1).indices.to(torch.int32).contiguous()
    hist_pred = torch.bincount(pred_idx.reshape(-1).long(), minlength=E).to(torch.int32)
    res = {}
    for how in ("none", "hist", "hist_plan", "slot_expert", "slot_quota"):
        for end in (False, True):
            layer = MoELayer(cfg)
            layer.set_weights(*ws)
            given = logits.clone()
            if how != "none":
                flat = given.view(torch.int32).reshape(-1)
                n = getattr(layer, how).numel()
                setattr(layer, how, flat[-n:] if end else flat[:n])
            assert layer._one_call(given, x, hist_pred, pred_idx, mode)
            res[how, end] = outputs(layer)
    for how, got in res.items():
        for n, v in res["none", False].items():
            assert torch.equal(got[n], v), (how, n)
