"""GPU parity of the grouped SwiGLU FFN and of the whole layer against the fp64 oracle.

Tolerances: max|delta| <= 1e-5 * max|ref| for fp32 and <= 2e-2 * max|ref| for bf16
storage with fp32 accumulation (hidden activation and output rounded to bf16)."""
import numpy as np
import pytest
import torch

from oracle import grouped_ffn, ffn_rows, combine, moe_layer
from oracle.histogram import skewness
from oracle.ffn import ffn_rows_relu
from paper_2506_07366_amd import binding as B
from paper_2506_07366_amd import workloads as wl
from paper_2506_07366_amd.layer import MoELayer, to_device
from gpu_util import Case, dev_i32, to_host_f32, weights_storage, shape_key

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


@pytest.fixture
def ffn_options():
    """Sets overrides of the grouped FFN's automatic choices and restores the defaults afterwards."""
    def set_(tile1=-1, tile2=-1, split=-1, group_n=0):
        B.moe_grouped_ffn_set_option(B.FFN_OPT_TILE1, tile1)
        B.moe_grouped_ffn_set_option(B.FFN_OPT_TILE2, tile2)
        B.moe_grouped_ffn_set_option(B.FFN_OPT_SPLIT_K, split)
        B.moe_grouped_ffn_set_option(B.FFN_OPT_GROUP_N, group_n)
    yield set_
    set_()


def expert_row_lists(seg_offsets, slot_expert, E):
    """Rows of x_perm per expert in the order the FFN tiles them: segments of the expert in
    ascending slot id, rows ascending."""
    lists = [[] for _ in range(E)]
    for s_, e in enumerate(slot_expert):
        if 0 <= e < E:
            lists[e].extend(range(int(seg_offsets[s_]), int(seg_offsets[s_ + 1])))
    return lists


def host_weights(cfg):
    W1s, W3s, W2s = weights_storage(shape_key(cfg))
    return W1s, W3s, W2s


def dev_weights(cfg, Ws):
    return tuple(to_device(w, cfg.dtype) for w in Ws)


def rel_err(got, ref):
    return float(np.max(np.abs(got - ref)) / max(np.max(np.abs(ref)), 1e-30))


def run_ffn_case(cfg, seg_sizes, slot_expert, seed=0):
    """x_perm with the given ragged segments through the HIP FFN and the oracle."""
    rng = np.random.default_rng(seed)
    A = int(sum(seg_sizes))
    x = wl.quantize(rng.standard_normal((A, cfg.d)).astype(np.float32), cfg.dtype)
    seg_offsets = np.concatenate([[0], np.cumsum(seg_sizes)]).astype(np.int32)
    Ws = host_weights(cfg)
    packed = B.moe_pack_weights(*dev_weights(cfg, Ws))
    y = B.moe_grouped_ffn(to_device(wl.to_storage(x, cfg.dtype), cfg.dtype), dev_i32(seg_offsets),
                          dev_i32(slot_expert), packed, cfg.E, cfg.ffn)
    Wf = [wl.from_storage(w, cfg.dtype) for w in Ws]
    ref = grouped_ffn(x, seg_offsets, slot_expert, *Wf)
    return to_host_f32(y), ref, seg_offsets


@pytest.mark.parametrize("dtype,d,ffn", [("f32", 128, 256), ("f32", 36, 20), ("bf16", 128, 256), ("bf16", 512, 1024),
                                         ("bf16", 64, 64), ("bf16", 192, 1408), ("bf16", 128, 688), ("bf16", 64, 20),
                                         ("bf16", 256, 1376)])
def test_ffn_ragged_segments(dtype, d, ffn):
    E = 5
    cfg = wl.MoEConfig("f", T=1, d=d, ffn=ffn, E=E, k=1, G=4, S=3, dtype=dtype, mode=0, seed=21)
    # sizes around the tile edges (64/128/256) and empty segments; an empty slot (-1) with no rows
    seg_sizes = [1, 0, 127, 129, 0, 256, 257, 63, 300, 0, 5, 64]
    slot_expert = [0, 1, 2, 3, -1, 4, 0, 1, 2, 3, 4, 0]
    got, ref, so = run_ffn_case(cfg, seg_sizes, slot_expert)
    assert rel_err(got, ref) <= TOL[dtype]
    # per-row check too (a wrong expert or a dropped tail row must not hide behind the global max)
    scale = np.max(np.abs(ref))
    assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL[dtype] * scale)


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("d,ffn,scale", [(4, 4, 1),       # one quarter of a 16-deep step, four columns
                                         (20, 68, 1),     # ragged steps and columns, 32-row tiles
                                         (144, 260, 1),   # nine steps (chunks of four), one column tile of four columns
                                         (36, 2052, 12)]) # enough tiles for the 64-row form
def test_ffn_f32_tile_edges(d, ffn, scale, relu):
    """fp32 products at row counts around the 32- and 64-row tiles and at widths that are no multiple
    of a step or a column tile.  An expert without rows holds inf and nan: nothing of it may show."""
    cfg = wl.CONFIGS["cfg1_tiny_f32"].replace(d=d, ffn=ffn, seed=17)
    sizes = [r * scale for r in (1, 31, 32, 33, 0, 64, 65, 127, 2, 0, 63, 16)]
    slot_expert = np.array([0, 1, 2, 3, 4, 5, 6, 7, 0, -1, 1, 6], dtype=np.int32)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    rng = np.random.default_rng(3)
    x = rng.standard_normal((int(offs[-1]), d)).astype(np.float32)
    W1, W3, W2 = [w.copy() for w in host_weights(cfg)]
    for w in (W1, W3, W2):
        w[4] = np.inf
        w[4, ::2] = np.nan
    dx, so, se = torch.from_numpy(x).cuda(), dev_i32(offs), dev_i32(slot_expert)
    if relu:
        packed = B.moe_pack_weights_relu(*[to_device(w, "f32") for w in (W1, W2)])
    else:
        packed = B.moe_pack_weights(*[to_device(w, "f32") for w in (W1, W3, W2)])
    y = to_host_f32(B.moe_grouped_ffn(dx, so, se, packed, cfg.E, ffn, relu=relu))
    ref = np.zeros((x.shape[0], d))
    for s_, e in enumerate(slot_expert):
        lo, hi = offs[s_], offs[s_ + 1]
        if hi > lo:
            ref[lo:hi] = ffn_rows_relu(x[lo:hi], W1[e], W2[e]) if relu else ffn_rows(x[lo:hi], W1[e], W3[e], W2[e])
    assert rel_err(y, ref) <= TOL["f32"]


def test_ffn_pack_and_f32_rows_at_any_address():
    """Weights packed from, and fp32 rows read and written at, addresses that only suit their element
    type: the same bytes as from aligned tensors."""
    def shifted(t, by):
        room = torch.zeros(t.numel() + by, dtype=t.dtype, device="cuda")
        room[by:] = t.flatten()
        return room[by:].view(t.shape)

    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    E, d, ffn, A = 3, 64, 72, 50
    so, se = dev_i32([0, 20, 30, A]), dev_i32([0, 2, 1])
    for dtype in (torch.bfloat16, torch.float32):
        W = [torch.randn(sh, device="cuda", generator=g).to(dtype) for sh in ((E, d, ffn), (E, d, ffn), (E, ffn, d))]
        packed = B.moe_pack_weights(*W)
        if dtype == torch.bfloat16:
            for by in (1, 3, 4):
                assert torch.equal(packed, B.moe_pack_weights(*[shifted(w, by) for w in W]))
            continue
        x = torch.randn((A, d), device="cuda", generator=g)
        y = B.moe_grouped_ffn(x, so, se, packed, E, ffn)
        for by in (1, 2, 3):
            out = shifted(torch.zeros_like(x), by)
            assert torch.equal(y, B.moe_grouped_ffn(shifted(x, by), so, se, packed, E, ffn, out=out))


def test_ffn_slot_range_only_touches_its_rows():
    cfg = wl.MoEConfig("f", T=1, d=128, ffn=256, E=5, k=1, G=4, S=3, dtype="bf16", mode=0, seed=21)
    rng = np.random.default_rng(5)
    seg_sizes = [40, 0, 130, 7, 0, 200, 33, 0, 64, 1, 0, 90]
    slot_expert = [0, -1, 2, 3, -1, 4, 0, -1, 2, 3, -1, 1]
    A = sum(seg_sizes)
    x = wl.quantize(rng.standard_normal((A, cfg.d)).astype(np.float32), "bf16")
    so = np.concatenate([[0], np.cumsum(seg_sizes)]).astype(np.int32)
    Ws = host_weights(cfg)
    packed = B.moe_pack_weights(*dev_weights(cfg, Ws))
    xd = to_device(wl.to_storage(x, "bf16"), "bf16")
    y_full = B.moe_grouped_ffn(xd, dev_i32(so), dev_i32(slot_expert), packed, cfg.E, cfg.ffn)
    y_rank = B.moe_grouped_ffn(xd, dev_i32(so), dev_i32(slot_expert), packed, cfg.E, cfg.ffn, seg_begin=3, seg_end=6)
    yf, yr = to_host_f32(y_full), to_host_f32(y_rank)
    assert np.array_equal(yr[so[3]:so[6]], yf[so[3]:so[6]])
    assert np.all(yr[:so[3]] == 0) and np.all(yr[so[6]:] == 0)


@pytest.mark.parametrize("name", ["cfg1_tiny_f32", "mid_bf16"])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_layer_full_compare(name, mode):
    """Whole path on configs the oracle finishes in full."""
    cfg = wl.CONFIGS[name].replace(mode=mode, acc=0.9, sigma_pred=wl.CONFIGS[name].sigma_pred)
    case = Case(cfg)
    Ws = host_weights(cfg)
    Wf = [wl.from_storage(w, cfg.dtype) for w in Ws]
    ref = moe_layer(mode, case.logits, case.x, *Wf, cfg.k, cfg.G, cfg.S, cfg.cmax,
                    hist_pred=case.hist_plan, pred_idx=case.pred_idx)
    layer = MoELayer(cfg)
    layer.set_weights(*dev_weights(cfg, Ws))
    out = layer.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(), pred_idx=case.dev_pred_idx())
    torch.cuda.synchronize()
    assert np.array_equal(layer.topk_idx.cpu().numpy(), ref["topk_idx"])
    assert np.array_equal(layer.perm["row_of_assign"].cpu().numpy(), ref["perm"]["row_of_assign"])
    assert np.array_equal(layer.slot_expert.cpu().numpy(), ref["plan"].slot_expert)
    assert rel_err(to_host_f32(layer.y_perm), ref["y_perm"]) <= TOL[cfg.dtype]
    assert rel_err(to_host_f32(out), ref["out"]) <= TOL[cfg.dtype]
    rep = layer.load_report()
    assert rep["makespan"] == int(ref["perm"]["rank_load"].max())
    assert rep["n_iters"] == ref["plan"].n_iters
    assert rep["skewness"] == pytest.approx(skewness(ref["hist"] if "hist" in ref else case.hist), rel=1e-12)
    assert rep["imbalance"] == pytest.approx(float(ref["perm"]["rank_load"].max()) * cfg.G / cfg.A, rel=1e-12)


FULL = ["cfg2_mixtral_dist", "cfg3_mixtral_t2e", "cfg4_finegrained"] + \
       [f"cfg5_prefill_a{a}_m{m}" for a in ("0.1", "1", "10") for m in (0, 1, 2)] + \
       ["cfg5_decode_m0", "cfg5_decode_m1", "cfg5_decode_m2", "cfg6_switch_relu", "cfg7_llama_moe"]


@pytest.mark.parametrize("name", FULL)
def test_layer_full_size_sampled(name):
    """Full-size configs in the launch configuration the benchmark times: integer
    outputs compared in full, FFN / layer outputs on sampled rows the oracle can
    compute one by one: all k rows of sampled tokens, the first and last row of
    every non-empty segment, and the rows either side of every tile boundary the
    kernels can use (rows are tiled per expert, over all its segments, in tiles of
    some multiple of 32 rows: every multiple of 32 in every expert's row list).  The
    load report is compared with the oracle's skewness and rank loads."""
    cfg = wl.CONFIGS[name]
    case = Case(cfg)
    Ws = host_weights(cfg)
    layer = MoELayer(cfg)
    layer.set_weights(*dev_weights(cfg, Ws))
    out = layer.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(), pred_idx=case.dev_pred_idx())
    torch.cuda.synchronize()
    assert np.array_equal(layer.topk_idx.cpu().numpy(), case.idx)
    assert np.array_equal(layer.hist.cpu().numpy(), case.hist)
    assert np.array_equal(layer.slot_expert.cpu().numpy(), case.plan.slot_expert)
    assert np.array_equal(layer.slot_quota.cpu().numpy(), case.plan.slot_quota)
    assert np.array_equal(layer.perm["seg_offsets"].cpu().numpy(), case.perm["seg_offsets"])
    assert np.array_equal(layer.perm["row_of_assign"].cpu().numpy(), case.perm["row_of_assign"])
    assert np.array_equal(layer.perm["rank_load"].cpu().numpy(), case.perm["rank_load"])

    rng = np.random.default_rng(123)
    n_tok = min(cfg.T, 128)
    toks = np.sort(rng.choice(cfg.T, size=n_tok, replace=False))
    roa = case.perm["row_of_assign"].reshape(cfg.T, cfg.k)
    rows = set(roa[toks].reshape(-1).tolist())
    so = case.perm["seg_offsets"]
    for s in range(cfg.nseg):
        lo, hi = int(so[s]), int(so[s + 1])
        if hi > lo:
            rows.update([lo, hi - 1])
    for lst in expert_row_lists(so, case.plan.slot_expert, cfg.E):
        for b in range(32, len(lst), 32):         # every tile boundary inside the expert's rows
            rows.update([lst[b - 1], lst[b]])
    rows = np.array(sorted(rows), dtype=np.int64)
    aor = case.perm["assign_of_row"]
    seg_of_row = np.searchsorted(so, rows, side="right") - 1
    exp_of_row = case.plan.slot_expert[seg_of_row]
    assert np.array_equal(exp_of_row, case.idx.reshape(-1)[aor[rows]])
    y_ref = np.zeros((rows.size, cfg.d))
    for e in np.unique(exp_of_row):
        sel = np.nonzero(exp_of_row == e)[0]
        xr = case.x[aor[rows[sel]] // cfg.k]
        if cfg.act == "relu":
            y_ref[sel] = ffn_rows_relu(xr, wl.from_storage(Ws[0][e], cfg.dtype), wl.from_storage(Ws[2][e], cfg.dtype))
        else:
            y_ref[sel] = ffn_rows(xr, wl.from_storage(Ws[0][e], cfg.dtype), wl.from_storage(Ws[1][e], cfg.dtype),
                                  wl.from_storage(Ws[2][e], cfg.dtype))
    y_got = to_host_f32(layer.y_perm[torch.from_numpy(rows).cuda()])
    scale = np.max(np.abs(y_ref))
    assert np.all(np.max(np.abs(y_got - y_ref), axis=1) <= TOL[cfg.dtype] * scale)
    # layer output of the sampled tokens
    pos = {int(r): i for i, r in enumerate(rows)}
    out_ref = np.zeros((n_tok, cfg.d))
    for i, t in enumerate(toks):
        for j in range(cfg.k):
            out_ref[i] += case.w[t, j] * y_ref[pos[int(roa[t, j])]]
    out_got = to_host_f32(out[torch.from_numpy(toks).cuda()])
    assert np.max(np.abs(out_got - out_ref)) <= TOL[cfg.dtype] * np.max(np.abs(out_ref))
    # properties that hold at any size
    assert int(layer.perm["rank_load"].sum()) == cfg.A
    assert torch.isfinite(out.float()).all()
    # load report against the oracle: skewness of the histogram, bottleneck rank over the mean
    rep = layer.load_report()
    assert rep["skewness"] == pytest.approx(skewness(case.hist), rel=1e-12)
    assert rep["imbalance"] == pytest.approx(float(case.perm["rank_load"].max()) * cfg.G / cfg.A, rel=1e-12)
    assert rep["makespan"] == int(case.perm["rank_load"].max())
    assert rep["rank_load"] == case.perm["rank_load"].tolist()


def test_output_independent_of_plan_mode():
    """Replicas hold the same weights: the layer output must not depend on the plan."""
    cfg = wl.CONFIGS["mid_bf16"]
    Ws = host_weights(cfg)
    outs = []
    for mode in (0, 1, 2):
        c = cfg.replace(mode=mode, acc=0.8)
        case = Case(c)
        layer = MoELayer(c)
        layer.set_weights(*dev_weights(c, Ws))
        out = layer.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(),
                         pred_idx=case.dev_pred_idx())
        outs.append(to_host_f32(out))
    scale = np.max(np.abs(outs[0]))
    assert np.max(np.abs(outs[1] - outs[0])) <= 2e-2 * scale
    assert np.max(np.abs(outs[2] - outs[0])) <= 2e-2 * scale


def test_identity_round_trip_permute_combine():
    """permute then combine with y_perm := x_perm returns x (gate weights sum to 1)."""
    cfg = wl.MoEConfig("rt", T=777, d=256, ffn=64, E=16, k=4, G=4, S=6, dtype="f32", mode=1, sigma_pred=0.3, seed=6)
    case = Case(cfg)
    x = case.dev_x()
    idx, w = B.moe_route_topk(case.dev_logits(), cfg.k)
    out = B.moe_permute(1, x, idx, None, dev_i32(case.hist), case.dev_hist_plan(), dev_i32(case.plan.slot_expert),
                        dev_i32(case.plan.slot_quota), cfg.E, cfg.G, cfg.S)
    back = B.moe_combine(out["x_perm"], out["row_of_assign"], w, cfg.T, cfg.k)
    assert np.max(np.abs(to_host_f32(back) - case.x)) <= 1e-5 * np.max(np.abs(case.x))


@pytest.mark.parametrize("name,mode", [("cfg1_tiny_f32", 1), ("mid_bf16", 0), ("mid_bf16", 1), ("mid_bf16", 2),
                                       ("cfg4_finegrained", 1)])
def test_fused_gather_equals_copied_rows(name, mode):
    """Gathering the token rows inside the first product must give exactly what the
    FFN gives on the copied rows (same arithmetic on the same values)."""
    cfg = wl.CONFIGS[name].replace(mode=mode, acc=0.9)
    case = Case(cfg)
    Ws = host_weights(cfg)
    dw = dev_weights(cfg, Ws)
    outs = []
    for fused in (False, True):
        layer = MoELayer(cfg, fused_gather=fused)
        layer.set_weights(*dw)
        out = layer.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(),
                         pred_idx=case.dev_pred_idx())
        torch.cuda.synchronize()
        outs.append((layer.y_perm.float().cpu().numpy().copy(), out.float().cpu().numpy().copy()))
        assert np.array_equal(layer.perm["row_of_assign"].cpu().numpy(), case.perm["row_of_assign"])
    assert np.array_equal(outs[0][0], outs[1][0])
    assert np.array_equal(outs[0][1], outs[1][1])


def test_fused_gather_slot_range_and_oracle():
    cfg = wl.CONFIGS["mid_bf16"]
    case = Case(cfg)
    Ws = host_weights(cfg)
    Wf = [wl.from_storage(w, cfg.dtype) for w in Ws]
    layer = MoELayer(cfg, fused_gather=True)
    layer.set_weights(*dev_weights(cfg, Ws))
    layer.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(), pred_idx=None)
    x_perm = case.x[case.perm["assign_of_row"] // cfg.k]
    ref = grouped_ffn(x_perm, case.perm["seg_offsets"], case.plan.slot_expert, *Wf)
    assert rel_err(to_host_f32(layer.y_perm), ref) <= TOL["bf16"]
    # one rank's slots alone
    layer.y_perm.zero_()
    layer.ffn(seg_begin=cfg.S, seg_end=2 * cfg.S)
    so = case.perm["seg_offsets"]
    got = to_host_f32(layer.y_perm)
    lo, hi = so[cfg.S], so[2 * cfg.S]
    assert rel_err(got[lo:hi], ref[lo:hi]) <= TOL["bf16"]
    assert np.all(got[:lo] == 0) and np.all(got[hi:] == 0)


# ---------------------------------------------------------------- ReLU form of the FFN
@pytest.mark.parametrize("dtype,d,ffn", [("f32", 128, 256), ("f32", 36, 20), ("bf16", 128, 256), ("bf16", 512, 1024),
                                         ("bf16", 64, 64), ("bf16", 768, 3072), ("bf16", 192, 1408), ("bf16", 128, 688),
                                         ("bf16", 64, 8)])
def test_relu_ffn_ragged_segments(dtype, d, ffn):
    E = 5
    cfg = wl.MoEConfig("f", T=1, d=d, ffn=ffn, E=E, k=1, G=4, S=3, dtype=dtype, mode=0, seed=21, act="relu")
    seg_sizes = [1, 0, 127, 129, 0, 256, 257, 63, 300, 0, 5, 64]
    slot_expert = [0, 1, 2, 3, -1, 4, 0, 1, 2, 3, 4, 0]
    rng = np.random.default_rng(3)
    A = int(sum(seg_sizes))
    x = wl.quantize(rng.standard_normal((A, d)).astype(np.float32), dtype)
    seg_offsets = np.concatenate([[0], np.cumsum(seg_sizes)]).astype(np.int32)
    W1s, _, W2s = host_weights(cfg)
    packed = B.moe_pack_weights_relu(to_device(W1s, dtype), to_device(W2s, dtype))
    y = B.moe_grouped_ffn(to_device(wl.to_storage(x, dtype), dtype), dev_i32(seg_offsets), dev_i32(slot_expert),
                          packed, E, ffn, relu=True)
    ref = grouped_ffn(x, seg_offsets, slot_expert, wl.from_storage(W1s, dtype), None, wl.from_storage(W2s, dtype))
    got = to_host_f32(y)
    scale = np.max(np.abs(ref))
    assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL[dtype] * scale)
    # the SwiGLU entry point on the same rows gives something else: the two forms are not mixed up
    assert scale > 0


def test_relu_layer_top1_full_compare():
    """A small top-1 ReLU layer end to end against the oracle (every output element)."""
    cfg = wl.MoEConfig("switch_small", T=700, d=128, ffn=256, E=12, k=1, G=4, S=4, dtype="bf16", mode=1, alpha=0.3,
                       sigma_pred=0.2, seed=31, act="relu")
    case = Case(cfg)
    Ws = host_weights(cfg)
    layer = MoELayer(cfg)
    layer.set_weights(*dev_weights(cfg, Ws))
    out = layer.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(), pred_idx=None)
    ref = moe_layer(cfg.mode, case.logits, case.x, wl.from_storage(Ws[0], cfg.dtype), None,
                    wl.from_storage(Ws[2], cfg.dtype), cfg.k, cfg.G, cfg.S, cfg.cmax, hist_pred=case.hist_plan)
    assert np.array_equal(layer.perm["row_of_assign"].cpu().numpy(), ref["perm"]["row_of_assign"])
    assert rel_err(to_host_f32(layer.y_perm), ref["y_perm"]) <= TOL[cfg.dtype]
    assert rel_err(to_host_f32(out), ref["out"]) <= TOL[cfg.dtype]
    # top-1: the gate weight is exactly 1, the layer output is the expert output of the token's row
    assert np.all(case.w == 1.0)


def test_ffn_many_tiny_segments():
    """2048 segments (the limit) of 0..5 rows each: every M-tile is a ragged one."""
    rng = np.random.default_rng(8)
    E, d, ffn, nseg = 32, 64, 64, 2048
    cfg = wl.MoEConfig("tiny", T=1, d=d, ffn=ffn, E=E, k=1, G=256, S=8, dtype="bf16", mode=0, seed=23)
    seg_sizes = rng.integers(0, 6, size=nseg).tolist()
    slot_expert = [int(e) if n > 0 or rng.random() < 0.5 else -1 for e, n in zip(rng.integers(0, E, size=nseg), seg_sizes)]
    got, ref, so = run_ffn_case(cfg, seg_sizes, slot_expert, seed=9)
    scale = np.max(np.abs(ref))
    assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL["bf16"] * scale)


@pytest.mark.parametrize("split", [-1, 1])
def test_ffn_many_experts_full_and_ragged_tiles(split, ffn_options):
    """1024 experts (the limit) over 2048 segments, a few experts with several full-height tiles and
    several segments, the rest slivers: every expert's ragged tile has to find its place among a
    thousand others, with and without tiles split along K."""
    ffn_options(split=split)
    rng = np.random.default_rng(18)
    E, d, ffn, nseg = 1024, 64, 256, 2048
    cfg = wl.MoEConfig("many", T=1, d=d, ffn=ffn, E=E, k=1, G=256, S=8, dtype="bf16", mode=0, seed=24)
    seg_sizes = rng.integers(0, 4, size=nseg)
    slot_expert = rng.integers(0, E, size=nseg)
    big = rng.choice(nseg, size=12, replace=False)
    seg_sizes[big] = rng.integers(200, 700, size=12)
    slot_expert[big] = rng.integers(0, 5, size=12)          # several segments of the same few experts
    slot_expert = [int(e) if n > 0 or rng.random() < 0.5 else -1 for e, n in zip(slot_expert, seg_sizes)]
    got, ref, so = run_ffn_case(cfg, [int(n) for n in seg_sizes], slot_expert, seed=19)
    scale = np.max(np.abs(ref))
    assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL["bf16"] * scale)


@pytest.mark.parametrize("dtype,split", [("f32", -1), ("bf16", -1), ("bf16", 1)])
@pytest.mark.parametrize("E,nseg,rows", [(1, 1, 5), (63, 64, 3000), (65, 130, 3000), (1023, 2047, 5000), (1024, 2048, 5000)])
def test_ffn_tables_of_many_slots(E, nseg, rows, dtype, split, ffn_options):
    """Row list and tile tables where segments, experts and rows cross wavefronts and workgroups:
    replicas in any order, empty and unused slots, many ragged tiles of equal height."""
    ffn_options(split=split)
    rng = np.random.default_rng(E + nseg)
    cfg = wl.MoEConfig("f", T=1, d=64, ffn=128, E=E, k=1, G=1, S=E, dtype=dtype, mode=0, seed=9)
    slot_expert = rng.integers(-1, E, nseg).astype(np.int32)
    slot_expert[: min(E, nseg)] = rng.permutation(E)[: min(E, nseg)]
    rng.shuffle(slot_expert)
    p = np.where(slot_expert >= 0, rng.random(nseg) ** 4, 0)
    sizes = rng.multinomial(rows, p / p.sum()).tolist()
    got, ref, _ = run_ffn_case(cfg, sizes, slot_expert, seed=2)
    assert rel_err(got, ref) <= TOL[dtype]


@pytest.mark.parametrize("split", [-1, 1])
@pytest.mark.parametrize("E,nseg,live", [(257, 300, [256]), (512, 512, [0, 511]), (1024, 1024, [63, 64, 320, 1023]),
                                         (1000, 2048, [127, 128, 129, 999])])
def test_ffn_tables_few_experts_of_many(E, nseg, live, split, ffn_options):
    """Rows on a handful of experts at the ends of groups of 64: the groups without rows are skipped."""
    ffn_options(split=split)
    rng = np.random.default_rng(E)
    cfg = wl.MoEConfig("f", T=1, d=64, ffn=128, E=E, k=1, G=1, S=E, dtype="bf16", mode=0, seed=9)
    slot_expert = np.concatenate([np.arange(E), rng.integers(0, E, nseg - E)]).astype(np.int32)
    rng.shuffle(slot_expert)
    sizes = np.where(np.isin(slot_expert, live), rng.integers(0, 300, nseg), 0).tolist()
    sizes[int(np.flatnonzero(slot_expert == live[-1])[0])] = 65   # (one at least holds rows)
    got, ref, _ = run_ffn_case(cfg, sizes, slot_expert, seed=2)
    assert rel_err(got, ref) <= TOL["bf16"]


def test_ffn_one_huge_segment_and_empty_rest():
    """All rows in the last of 12 segments: 20 full-height tiles of one expert, nothing else."""
    cfg = wl.MoEConfig("huge", T=1, d=128, ffn=256, E=5, k=1, G=4, S=3, dtype="bf16", mode=0, seed=21)
    seg_sizes = [0] * 11 + [5120]
    slot_expert = [0, 1, 2, 3, -1, 4, 0, 1, 2, 3, 4, 2]
    got, ref, so = run_ffn_case(cfg, seg_sizes, slot_expert, seed=10)
    scale = np.max(np.abs(ref))
    assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL["bf16"] * scale)


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("tile2", [0, 1, 2])
@pytest.mark.parametrize("tile1", [0, 1, 2])
def test_ffn_every_tile_variant(tile1, tile2, split, ffn_options):
    """The tile shapes built into the library (forced through moe_grouped_ffn_set_option) all
    compute the same FFN, with the closing tiles of the second product computed whole (0) or as
    parts of K added up afterwards (1: forced; 320 hidden columns are 5 k-tiles, so the four
    parts are unequal)."""
    ffn_options(tile1=tile1, tile2=tile2, split=split)
    cfg = wl.MoEConfig("v", T=1, d=256, ffn=320, E=5, k=1, G=4, S=3, dtype="bf16", mode=0, seed=21)
    seg_sizes = [1, 0, 127, 129, 0, 256, 257, 63, 300, 0, 5, 64]
    slot_expert = [0, 1, 2, 3, -1, 4, 0, 1, 2, 3, 4, 0]
    got, ref, so = run_ffn_case(cfg, seg_sizes, slot_expert, seed=tile1 * 3 + tile2)
    scale = np.max(np.abs(ref))
    assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL["bf16"] * scale)


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("d,ffn", [(64, 128), (192, 256), (320, 384), (448, 576), (704, 832)])
def test_ffn_tile_heights_and_depths(d, ffn, relu, ffn_options):
    """Tiles of every height the kernel has a K loop for, at its edges, with every remainder of the
    number of k-tiles (1 to 13) by the three or four that are under way at a time."""
    ffn_options(tile1=0, tile2=0, split=0)
    sizes = [1, 31, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256, 256 + 40]
    E = len(sizes)
    cfg = wl.MoEConfig("h", T=1, d=d, ffn=ffn, E=E, k=1, G=E, S=1, dtype="bf16", mode=0, seed=47,
                       act="relu" if relu else "swiglu")
    A = sum(sizes)
    x = wl.quantize(np.random.default_rng(48).standard_normal((A, d)).astype(np.float32), "bf16")
    so = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    W1s, W3s, W2s = host_weights(cfg)
    Wf = [wl.from_storage(w, "bf16") for w in (W1s, W3s, W2s)]
    packed = B.moe_pack_weights_relu(to_device(W1s, "bf16"), to_device(W2s, "bf16")) if relu \
        else B.moe_pack_weights(*dev_weights(cfg, (W1s, W3s, W2s)))
    got = to_host_f32(B.moe_grouped_ffn(to_device(wl.to_storage(x, "bf16"), "bf16"), dev_i32(so), dev_i32(range(E)),
                                        packed, E, ffn, relu=relu))
    ref = grouped_ffn(x, so, list(range(E)), Wf[0], None if relu else Wf[1], Wf[2])
    assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL["bf16"] * np.max(np.abs(ref)))


@pytest.mark.parametrize("relu", [False, True])
def test_ffn_weights_read_past_the_caches(relu, ffn_options):
    """A layer whose weights are too large for the caches reads those of an expert's only M-tile past them,
    whatever its height: the same bits as the same experts in a small layer."""
    ffn_options(tile1=0, tile2=0, split=0)
    d, ffn, many = 512, 832, 170                   # W2 of 170 experts: 138 MiB; 8 and 13 k-tiles
    sizes = [1, 31, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256, 256 + 40]
    E, A = len(sizes), sum(sizes)
    gen = torch.Generator().manual_seed(51)
    w = [(torch.randn(E, *shape, generator=gen) * 0.05).to(torch.bfloat16).cuda()
         for shape in ([(d, ffn)] if relu else [(d, ffn), (d, ffn)]) + [(ffn, d)]]
    x = torch.randn(A, d, generator=gen).to(torch.bfloat16).cuda()
    so = dev_i32(np.concatenate([[0], np.cumsum(sizes)]))
    got = []
    for n in (E, many):
        # the small layer's experts are the large one's last
        packed = (B.moe_pack_weights_relu if relu else B.moe_pack_weights)(
            *[torch.cat([torch.zeros(n - E, *m.shape[1:], dtype=m.dtype, device=m.device), m]) for m in w])
        got.append(B.moe_grouped_ffn(x, so, dev_i32(range(n - E, n)), packed, n, ffn, relu=relu))
    assert torch.equal(got[0], got[1]) and torch.isfinite(got[0]).all() and got[0].any(dim=1).all()


@pytest.mark.parametrize("split", [-1, 0, 1])
@pytest.mark.parametrize("sizes", [
    [2049, 0, 2048, 1793, 257, 65],   # more and not more tiles than heights at 256 rows, a short last tile
    [1, 1, 1, 1, 1, 1],               # only short tiles
    [900, 899, 33, 64, 0, 129],       # tall and short ones, an expert without rows between
    [0, 0, 0, 0, 0, 3000]])           # one expert holds everything
def test_ffn_heights_chosen_from_the_batch(sizes, split, ffn_options):
    """Tables whose tile heights come from the rows per expert, every row present once: against the
    oracle, whole (four k-tiles are too few for the rule to split any) and all split along K.  Whole and split
    ones in one table: test_ffn_some_tiles_split_by_the_rule."""
    ffn_options(split=split)
    B.moe_grouped_ffn_set_option(B.FFN_OPT_STREAM, 0)
    try:
        cfg = wl.MoEConfig("c", T=1, d=128, ffn=256, E=6, k=1, G=3, S=3, dtype="bf16", mode=0, seed=49)
        slot_expert = [5, 1, -1, 0, 4, 5, 3, 2, 0]     # experts 0 and 5 in two slots each
        rows = dict(enumerate(sizes))
        seg = [rows[5] // 2, rows[1], 0, rows[0] - rows[0] // 3, rows[4], rows[5] - rows[5] // 2, rows[3], rows[2],
               rows[0] // 3]
        got, ref, _ = run_ffn_case(cfg, seg, slot_expert, seed=50)
        assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL["bf16"] * np.max(np.abs(ref)))
    finally:
        B.moe_grouped_ffn_set_option(B.FFN_OPT_STREAM, -1)


def second_table(ws, A, d, ffn, nseg):
    """Entries (first row, rows, expert, part, first, n_same) of the second product's M-tile table, and its counts of
    entries, whole tiles and split tiles, out of a workspace that a call has used."""
    up = lambda n: -(-n // 256) * 256
    head, cap = up(A * (-(-ffn // 64) * 64) * 2) + up(A * 4), -(-A // 32) + nseg
    # the sizes say how many split tiles there is room for (four parts each, 256 fp32 rows a part)
    split = next(n for n in range(1, 4096) if head + 2 * up((cap + 4 * n) * 32) + 256 + up(n * 8) + up(n * 4096 * d)
                 == B.moe_grouped_ffn_workspace_bytes(A, d, ffn, nseg, B.MOE_DTYPE_BF16))
    table = up((cap + 4 * split) * 32)
    raw = ws.cpu().numpy()
    entries, whole, splits = raw[head + 2 * table:][16:28].view(np.int32)
    return raw[head + table:][:32 * entries].view(np.int32).reshape(-1, 8)[:, [0, 1, 2, 5, 6, 7]], int(whole), int(splits)


@pytest.mark.parametrize("rows", [
    [540, 0, 123, 1467, 1116, 382],                                   # one tile split, of an expert with two
    [406, 753, 40, 1484, 51, 98, 638, 10, 410, 0, 281, 306]])         # the eight last ones of 24
def test_ffn_some_tiles_split_by_the_rule(rows, ffn_options):
    """Heights from the batch and the rule that splits the closing tiles, together: a table of whole tiles and of
    parts, the walk over an expert's whole tiles ends in front of its split ones, and a tile that shares its
    weights with them does not pass for the expert's only one.  Results against 64 bits."""
    ffn_options()
    d, ffn, E, A = 4096, 1024, len(rows), sum(rows)
    nseg = E + 3
    gen = torch.Generator(device="cuda").manual_seed(71)
    W1, W3, W2 = [torch.randn((E, *shape), device="cuda", generator=gen).mul_(0.03).to(torch.bfloat16)
                  for shape in ((d, ffn), (d, ffn), (ffn, d))]
    x = torch.randn((A, d), device="cuda", generator=gen).to(torch.bfloat16)
    offsets = np.concatenate([[0], np.cumsum(rows + [0, 0, 0])])
    ws = torch.zeros(B.moe_grouped_ffn_workspace_bytes(A, d, ffn, nseg, B.MOE_DTYPE_BF16), dtype=torch.uint8, device="cuda")
    y = B.moe_grouped_ffn(x, dev_i32(offsets), dev_i32([*range(E), -1, -1, -1]), B.moe_pack_weights(W1, W3, W2), E, ffn,
                          workspace=ws)
    ref = torch.cat([(torch.nn.functional.silu(v @ W1[e].double()) * (v @ W3[e].double())) @ W2[e].double()
                     for e, v in enumerate(x.double().split(rows))])
    assert float((y.double() - ref).abs().max()) <= TOL["bf16"] * float(ref.abs().max())
    table, n_whole, n_split = second_table(ws, A, d, ffn, nseg)
    assert n_whole > 0 and n_split > 0 and len(table) == n_whole + 4 * n_split
    tiles = table[:n_whole + n_split]                                 # (the first part of every split tile)
    covered = np.concatenate([np.arange(lo, lo + n) for lo, n in tiles[:, :2]])
    assert np.array_equal(np.sort(covered), np.arange(A))
    per_expert = np.bincount(tiles[:, 2], minlength=E)
    assert any(0 < np.sum(tiles[:n_whole, 2] == e) < per_expert[e] for e in range(E))
    for t, (_, _, e, part, first, n_same) in enumerate(table[:n_whole].tolist()):
        assert part == (-2 if per_expert[e] == 1 else -1)
        assert first <= t < first + n_same <= n_whole and np.all(table[first:first + n_same, 2] == e)


@pytest.mark.parametrize("form", [1, 2])
@pytest.mark.parametrize("d,ffn,relu", [(64, 64, False),      # one k-tile: one half / three parts of K are empty
                                        (192, 320, False),    # odd numbers of k-tiles, half a unit at the edge of N
                                        (576, 1088, True),    # nine and seventeen k-tiles, ReLU
                                        (2176, 192, False)])  # K above and below 32 k-tiles
def test_ffn_streaming_forms(form, d, ffn, relu):
    """The weight-streaming kernels at every count of 16-row groups, with M-tiles of one expert behind
    each other, empty slots and more experts than rows, in place and through the row gather with
    gate weights: against the oracle (bf16 tolerance of this file), the same bits twice and from a
    launch over a part of the slots."""
    _check_streaming(form, 6, d, ffn, relu)


@pytest.mark.parametrize("E,d,ffn,relu", [
    # up to 8 rows per expert on average and few columns: units of 32 columns, eight parts of K
    (46, 64, 64, False),      # one k-tile: seven parts of K are empty
    (46, 2176, 320, False),   # 34 k-tiles under gate and up columns
    (46, 576, 2176, False),   # and in the second product, nine in the first
    (46, 2176, 704, True),    # and under ReLU
    # more rows per expert: units of 64 columns, eight parts of a K above 32 k-tiles
    (6, 192, 2176, False),    # in the second product
    (6, 2176, 192, True)])    # and under ReLU
def test_ffn_streaming_first_form_units(E, d, ffn, relu):
    """The kernels of the first streaming form that the smallest batches take, with all eight wavefronts
    holding part of K."""
    _check_streaming(1, E, d, ffn, relu)


def _check_streaming(form, E, d, ffn, relu):
    cfg = wl.MoEConfig("s", T=1, d=d, ffn=ffn, E=E, k=1, G=4, S=3, dtype="bf16", mode=0, seed=41,
                       act="relu" if relu else "swiglu")
    seg_sizes = [1, 0, 16, 17, 0, 33, 64, 65, 130, 0, 5, 31]
    slot_expert = [0, 1, 2, 3, -1, 4, 0, 1, 2, -1, 4, 3]     # the last experts have no slot
    A = sum(seg_sizes)
    rng = np.random.default_rng(43)
    x = wl.quantize(rng.standard_normal((A, d)).astype(np.float32), "bf16")
    so = np.concatenate([[0], np.cumsum(seg_sizes)]).astype(np.int32)
    W1s, W3s, W2s = host_weights(cfg)
    Wf = [wl.from_storage(w, "bf16") for w in (W1s, W3s, W2s)]
    packed = B.moe_pack_weights_relu(to_device(W1s, "bf16"), to_device(W2s, "bf16")) if relu \
        else B.moe_pack_weights(*dev_weights(cfg, (W1s, W3s, W2s)))
    ref = grouped_ffn(x, so, slot_expert, Wf[0], None if relu else Wf[1], Wf[2])
    scale = np.max(np.abs(ref))
    xd = to_device(wl.to_storage(x, "bf16"), "bf16")
    args = (dev_i32(so), dev_i32(slot_expert), packed, E, ffn)
    try:
        B.moe_grouped_ffn_set_option(B.FFN_OPT_STREAM, form)
        y = B.moe_grouped_ffn(xd, *args, relu=relu)
        assert torch.equal(y, B.moe_grouped_ffn(xd, *args, relu=relu))
        part = B.moe_grouped_ffn(xd, *args, seg_begin=5, seg_end=9, relu=relu)
        got = to_host_f32(y)
        assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL["bf16"] * scale)
        assert np.array_equal(to_host_f32(part)[so[5]:so[9]], got[so[5]:so[9]])
        assert np.all(to_host_f32(part)[:so[5]] == 0) and np.all(to_host_f32(part)[so[9]:] == 0)
        if not relu:
            a_of_row = rng.permutation(A).astype(np.int32)
            src = np.empty_like(x)
            src[a_of_row] = x
            w = rng.random((A, 1)).astype(np.float32)
            yw = B.moe_grouped_ffn_gather(to_device(wl.to_storage(src, "bf16"), "bf16"), dev_i32(a_of_row), 1, *args,
                                          topk_w=torch.from_numpy(w).cuda())
            assert np.max(np.abs(to_host_f32(yw) - ref * w[a_of_row])) <= TOL["bf16"] * scale
    finally:
        B.moe_grouped_ffn_set_option(B.FFN_OPT_STREAM, -1)


def _order_sensitive(E, d, ffn, A, nseg, rows_on, seed):
    """A bf16 batch whose sums show the order they were taken in: every term of a product has its
    negative somewhere in the other half of K, so that what is left is rounding of the partial sums."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    r = lambda *shape: torch.randn(shape, device="cuda", generator=g).bfloat16()
    p = torch.randperm(d // 2, device="cuda", generator=g)
    q = torch.randperm(ffn // 2, device="cuda", generator=g)
    u, gate, up, down = r(A, d // 2), r(E, d // 2, ffn // 2), r(E, d, ffn // 2), r(E, ffn // 2, d)
    x = torch.cat([u, u[:, p]], 1)
    W1 = torch.cat([gate, -gate[:, p]], 1)
    W1, W3 = (torch.cat([w, w[:, :, q]], 2).contiguous() for w in (W1, up))   # hidden columns come in equal pairs
    packed = B.moe_pack_weights(W1, W3, torch.cat([down, -down[:, q]], 1))
    sizes = np.zeros(nseg, dtype=np.int64)
    sizes[:rows_on] = A // rows_on
    sizes[0] += A - sizes.sum()
    return x, dev_i32(np.concatenate([[0], np.cumsum(sizes)])), dev_i32(np.arange(nseg) % E), packed, E, ffn


@pytest.mark.parametrize("E,d,ffn,A,form1,form2", [
    (4, 512, 512, 16, 1, 1), (4, 512, 512, 64, 1, 1), (4, 512, 512, 65, 2, 2),   # up to 16 rows per expert; above
    (4, 512, 512, 256, 2, 2), (4, 512, 512, 257, 0, 0),         # up to 64 while tiles do not go once round
    (128, 512, 512, 256, 1, 1), (128, 512, 512, 257, 2, 2),     # small batches of up to 4 rows per expert
    (128, 512, 512, 2048, 2, 2), (128, 512, 512, 2049, 0, 0),   # short K: up to 16
    (32, 1088, 1088, 768, 2, 2), (32, 1088, 1088, 769, 0, 2),   # 24 rows per expert; the second product's tiles go once round
    (4, 512, 4224, 64, 1, 1), (4, 512, 4224, 65, 2, 0),         # 66 k-tiles in the second product
    (32, 1088, 6912, 545, 2, 0), (32, 1088, 7040, 545, 0, 0),   # 270 and 275 tiles of 17 k-tiles in the first product
    (1024, 2048, 1088, 14336, 2, 2), (1024, 2048, 1088, 14592, 0, 2),   # 126 and 128.25 k-tiles per CU in the first
])
def test_ffn_streaming_rule(E, d, ffn, A, form1, form2, ffn_options):
    """Which batches stream their weights: the automatic choice gives the bits of the form it is meant to
    be, on inputs where each form of either product gives its own."""
    args = _order_sensitive(E, d, ffn, A, E, min(E, 3), seed=A)

    def run(stream, tile1=-1, tile2=-1):
        ffn_options(tile1=tile1, tile2=tile2)
        B.moe_grouped_ffn_set_option(B.FFN_OPT_STREAM, stream)
        return B.moe_grouped_ffn(*args)

    try:
        forms = {(0, 0): run(0), (1, 1): run(1), (2, 2): run(2), (2, 0): run(2, tile2=1), (0, 2): run(2, tile1=1)}
        auto = run(-1)
    finally:
        B.moe_grouped_ffn_set_option(B.FFN_OPT_STREAM, -1)
    assert not any(torch.equal(forms[f], forms[h]) for f in forms for h in forms if f < h)
    assert torch.equal(auto, forms[form1, form2])


@pytest.mark.parametrize("relu", [False, True])
def test_ffn_split_k_matches_whole_tiles(relu, ffn_options):
    """Closing tiles computed as parts of K: same result as whole tiles up to the fp32
    association of the partial sums (one bf16 rounding step of the output), rows outside the
    slot range untouched, and the same answer on a second run (the order in which workgroups
    claim tiles does not reach the result)."""
    cfg = wl.MoEConfig("s", T=1, d=192, ffn=688, E=4, k=1, G=4, S=3, dtype="bf16", mode=0, seed=29)
    rng = np.random.default_rng(31)
    seg_sizes = [300, 0, 256, 1, 513, 0, 77, 255, 128, 0, 31, 640]
    slot_expert = [0, -1, 2, 3, 1, 2, 0, 1, 2, -1, 3, 0]
    A = sum(seg_sizes)
    x = wl.quantize(rng.standard_normal((A, cfg.d)).astype(np.float32), "bf16")
    so = np.concatenate([[0], np.cumsum(seg_sizes)]).astype(np.int32)
    W1s, W3s, W2s = host_weights(cfg)
    if relu:
        packed = B.moe_pack_weights_relu(to_device(W1s, "bf16"), to_device(W2s, "bf16"))
    else:
        packed = B.moe_pack_weights(*dev_weights(cfg, (W1s, W3s, W2s)))
    xd = to_device(wl.to_storage(x, "bf16"), "bf16")
    out = {}
    for split in (0, 1):
        ffn_options(split=split)
        out[split] = to_host_f32(B.moe_grouped_ffn(xd, dev_i32(so), dev_i32(slot_expert), packed, cfg.E, cfg.ffn,
                                                   relu=relu))
        again = to_host_f32(B.moe_grouped_ffn(xd, dev_i32(so), dev_i32(slot_expert), packed, cfg.E, cfg.ffn,
                                              relu=relu))
        assert np.array_equal(out[split], again)
        out[split, "range"] = to_host_f32(B.moe_grouped_ffn(xd, dev_i32(so), dev_i32(slot_expert), packed, cfg.E,
                                                            cfg.ffn, seg_begin=3, seg_end=8, relu=relu))
    Wf = [wl.from_storage(w, "bf16") for w in (W1s, W3s, W2s)]
    ref = grouped_ffn(x, so, slot_expert, Wf[0], None if relu else Wf[1], Wf[2])
    scale = np.max(np.abs(ref))
    for split in (0, 1):
        assert np.all(np.max(np.abs(out[split] - ref), axis=1) <= TOL["bf16"] * scale)
        r = out[split, "range"]
        assert np.max(np.abs(r[so[3]:so[8]] - ref[so[3]:so[8]])) <= TOL["bf16"] * scale
        assert np.all(r[:so[3]] == 0) and np.all(r[so[8]:] == 0)
    # whole (unsplit) tiles accumulate a row's products in the same order whatever else is launched
    # with them: the slot range alone gives the same bits as the full launch
    assert np.array_equal(out[0, "range"][so[3]:so[8]], out[0][so[3]:so[8]])
    assert np.max(np.abs(out[0] - out[1])) <= 2.0 ** -7 * scale


def test_ffn_replicas_of_one_expert_share_tiles():
    """Several segments of the range host the same expert (replicas hold the same weights):
    their rows are tiled together, whatever their sizes, and every row still gets its own
    expert's result; a row's result does not depend on which replica served it."""
    cfg = wl.MoEConfig("r", T=1, d=128, ffn=256, E=4, k=1, G=6, S=2, dtype="bf16", mode=0, seed=37)
    seg_sizes = [3, 200, 0, 58, 130, 1, 256, 7, 0, 90, 511, 2]
    slot_expert = [0, 1, 0, 0, 2, 0, 1, 0, -1, 3, 0, 1]      # expert 0 in seven slots, one of them empty
    got, ref, so = run_ffn_case(cfg, seg_sizes, slot_expert, seed=12)
    scale = np.max(np.abs(ref))
    assert np.all(np.max(np.abs(got - ref), axis=1) <= TOL["bf16"] * scale)
    # the same rows with every segment on its own (one launch per slot): same values up to the
    # position of the rows inside their tiles, which does not change a row's sum
    rng = np.random.default_rng(12)
    x = wl.quantize(rng.standard_normal((int(sum(seg_sizes)), cfg.d)).astype(np.float32), "bf16")
    Ws = host_weights(cfg)
    packed = B.moe_pack_weights(*dev_weights(cfg, Ws))
    xd = to_device(wl.to_storage(x, "bf16"), "bf16")
    y = torch.zeros_like(xd)
    for s_ in range(len(seg_sizes)):
        B.moe_grouped_ffn(xd, dev_i32(so), dev_i32(slot_expert), packed, cfg.E, cfg.ffn, seg_begin=s_, seg_end=s_ + 1,
                          out=y)
    assert np.array_equal(to_host_f32(y), got)


@pytest.mark.parametrize("name,mode", [("cfg1_tiny_f32", 1), ("mid_bf16", 0), ("mid_bf16", 1), ("mid_bf16", 2)])
def test_fused_gate_weights_against_oracle(name, mode):
    """Gate weights applied by the second product (moe_grouped_ffn_fused) and a plain sum in
    moe_combine: the layer output against the oracle's combine of the oracle's FFN, and the
    weighted rows against w * (oracle row).  Rule for the bits: fp32 rows are exactly
    fl(w * y) of the unweighted path's y; bf16 rows are rounded once from w * (fp32 sum), so
    they differ from bf16(w * bf16(y)) by at most one rounding step."""
    cfg = wl.CONFIGS[name].replace(mode=mode, acc=0.9)
    case = Case(cfg)
    Ws = host_weights(cfg)
    Wf = [wl.from_storage(w, cfg.dtype) for w in Ws]
    ref = moe_layer(mode, case.logits, case.x, *Wf, cfg.k, cfg.G, cfg.S, cfg.cmax,
                    hist_pred=case.hist_plan, pred_idx=case.pred_idx)
    dw = dev_weights(cfg, Ws)
    plain = MoELayer(cfg, fused_gather=True)
    plain.set_weights(*dw)
    plain.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(), pred_idx=case.dev_pred_idx())
    fused = MoELayer(cfg, fused_weights=True)
    fused.set_weights(*dw)
    out = fused.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(), pred_idx=case.dev_pred_idx())
    torch.cuda.synchronize()
    assert rel_err(to_host_f32(out), ref["out"]) <= TOL[cfg.dtype]
    w_row = case.w.reshape(-1)[ref["perm"]["assign_of_row"]]                 # gate weight of every row
    yw_ref = ref["y_perm"] * w_row[:, None]
    yw = to_host_f32(fused.y_perm)
    assert np.max(np.abs(yw - yw_ref)) <= TOL[cfg.dtype] * np.max(np.abs(ref["y_perm"]))
    y_plain = to_host_f32(plain.y_perm)
    w32 = fused.topk_w.cpu().numpy().reshape(-1)[ref["perm"]["assign_of_row"]].astype(np.float32)
    if cfg.dtype == "f32":
        assert np.array_equal(yw, y_plain * w32[:, None])
    else:
        twice = wl.quantize(y_plain * w32[:, None], "bf16")                  # rounded twice: bf16(w * bf16(sum))
        step = np.maximum(np.abs(yw), np.abs(twice)) * 2.0 ** -7             # a bf16 rounding step at that size
        assert np.all(np.abs(yw - twice) <= 2 * step + 1e-30)


def test_fused_gate_weights_full_size_sampled():
    """The fused path (row gather in the first product, gate weights in the second, plain sum
    in the combine) at the headline size: layer output of sampled tokens against the oracle."""
    cfg = wl.CONFIGS["cfg2_mixtral_dist"]
    case = Case(cfg)
    Ws = host_weights(cfg)
    layer = MoELayer(cfg, fused_weights=True)
    layer.set_weights(*dev_weights(cfg, Ws))
    out = layer.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(), pred_idx=case.dev_pred_idx())
    torch.cuda.synchronize()
    assert np.array_equal(layer.perm["row_of_assign"].cpu().numpy(), case.perm["row_of_assign"])
    rng = np.random.default_rng(77)
    toks = np.sort(rng.choice(cfg.T, size=96, replace=False))
    out_ref = np.zeros((toks.size, cfg.d))
    for i, t in enumerate(toks):
        for j in range(cfg.k):
            e = int(case.idx[t, j])
            y = ffn_rows(case.x[t:t + 1], wl.from_storage(Ws[0][e], cfg.dtype), wl.from_storage(Ws[1][e], cfg.dtype),
                         wl.from_storage(Ws[2][e], cfg.dtype))
            out_ref[i] += case.w[t, j] * y[0]
    out_got = to_host_f32(out[torch.from_numpy(toks).cuda()])
    assert np.max(np.abs(out_got - out_ref)) <= TOL["bf16"] * np.max(np.abs(out_ref))


@pytest.mark.parametrize("split", [-1, 1])
def test_ffn_workspace_exact_size_accepted_one_byte_less_refused(split, ffn_options):
    """The size moe_grouped_ffn_workspace_bytes reports is what the call needs: a caller-owned
    workspace of exactly that size works, one byte less is refused before anything is launched."""
    ffn_options(split=split)
    cfg = wl.MoEConfig("w", T=1, d=128, ffn=256, E=3, k=1, G=2, S=2, dtype="bf16", mode=0, seed=33)
    rng = np.random.default_rng(34)
    seg_sizes = [70, 300, 0, 129]
    slot_expert = [0, 1, -1, 2]
    A = sum(seg_sizes)
    x = wl.quantize(rng.standard_normal((A, cfg.d)).astype(np.float32), "bf16")
    so = np.concatenate([[0], np.cumsum(seg_sizes)]).astype(np.int32)
    Ws = host_weights(cfg)
    packed = B.moe_pack_weights(*dev_weights(cfg, Ws))
    xd = to_device(wl.to_storage(x, "bf16"), "bf16")
    need = B.moe_grouped_ffn_workspace_bytes(A, cfg.d, cfg.ffn, len(seg_sizes), 1)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    y = to_host_f32(B.moe_grouped_ffn(xd, dev_i32(so), dev_i32(slot_expert), packed, cfg.E, cfg.ffn, workspace=ws))
    Wf = [wl.from_storage(w, "bf16") for w in Ws]
    ref = grouped_ffn(x, so, slot_expert, *Wf)
    assert np.all(np.max(np.abs(y - ref), axis=1) <= TOL["bf16"] * np.max(np.abs(ref)))
    with pytest.raises(B.MoeGpsError):
        B.moe_grouped_ffn(xd, dev_i32(so), dev_i32(slot_expert), packed, cfg.E, cfg.ffn, workspace=ws[:need - 1])


def test_ffn_bits_do_not_depend_on_the_order_tiles_are_claimed():
    """Workgroups claim tiles from counters, so the order varies from run to run; a row's sums
    do not: ten runs of a Mixtral-shaped batch give the same bytes, split tiles included."""
    cfg = wl.CONFIGS["cfg2_mixtral_dist"].replace(T=1024)
    case = Case(cfg)
    Ws = host_weights(cfg)
    layer = MoELayer(cfg)
    layer.set_weights(*dev_weights(cfg, Ws))
    first = None
    for _ in range(10):
        out = layer.step(case.dev_logits(), case.dev_x(), hist_pred=case.dev_hist_plan(), pred_idx=case.dev_pred_idx())
        torch.cuda.synchronize()
        got = (layer.y_perm.view(torch.int16).clone(), out.view(torch.int16).clone())
        if first is None:
            first = got
        assert torch.equal(got[0], first[0]) and torch.equal(got[1], first[1])


@pytest.mark.parametrize("name,mode", [("mid_bf16", 1), ("mid_bf16", 2), ("cfg1_tiny_f32", 1)])
def test_layer_step_replays_from_a_hip_graph(name, mode):
    """The whole step captured into a HIP graph: every replay gives the eager step's bytes, also
    after the inputs were overwritten in place and with eager work and synchronisations between
    the replays."""
    cfg = wl.CONFIGS[name].replace(mode=mode, acc=0.9)
    case = Case(cfg)
    Ws = host_weights(cfg)
    dw = dev_weights(cfg, Ws)
    logits, x = case.dev_logits(), case.dev_x()
    hp, pi = case.dev_hist_plan(), case.dev_pred_idx()
    eager = MoELayer(cfg)
    eager.set_weights(*dw)
    layer = MoELayer(cfg)
    layer.set_weights(*dw)
    graph = layer.capture(logits, x, hist_pred=hp, pred_idx=pi)
    rng = np.random.default_rng(5)
    for rep in range(4):
        if rep > 0:   # new token rows and router logits in the captured tensors
            x.copy_(to_device(wl.to_storage(wl.quantize(rng.standard_normal((cfg.T, cfg.d)).astype(np.float32), cfg.dtype),
                                            cfg.dtype), cfg.dtype))
            logits.copy_(torch.from_numpy(rng.standard_normal((cfg.T, cfg.E)).astype(np.float32)).cuda())
        layer.out.zero_()
        layer.y_perm.zero_()
        torch.cuda.synchronize()
        graph.replay()
        ref = eager.step(logits, x, hist_pred=hp, pred_idx=pi)
        torch.cuda.synchronize()
        assert torch.equal(layer.topk_idx, eager.topk_idx)
        assert torch.equal(layer.perm["row_of_assign"], eager.perm["row_of_assign"])
        assert torch.equal(layer.out.view(torch.uint8), ref.view(torch.uint8)), rep


# width, hidden width of the SwiGLU and of the ReLU form, rows per expert, whether both products share a launch
# (tests/test_layer_step_launches.py holds the last against what is launched)
ONE_LAUNCH = [
    (768, 1700, 3400, [4000, 0, 0, 0, 0, 0, 0, 0], True),                  # one expert: the second product waits for all of the first
    (768, 1700, 3400, [1, 300, 0, 257, 1900, 64, 65, 1413], True),         # ragged, an expert without rows between, padded hidden width
    (832, 3200, 4000, [31, 33, 1700, 1, 2, 500, 129, 604], True),          # 13 k-tiles; 25 N-tiles; a round of tiles in the ReLU form
    (1024, 4000, 4000, [1500, 1501, 1502, 1503, 0, 1, 1000, 993], True),   # several rounds; 63 k-tiles in the second product
    (768, 1500, 3000, [200 + 7 * i for i in range(64)], True),             # many experts, between six and seven rounds
    (768, 5632, 5632, [700, 580], False), (768, 5632, 5632, [5000, 4472], False),   # 88 k-tiles in the second product
]


@pytest.mark.parametrize("form", ["plain", "relu", "gather", "weights"])
@pytest.mark.parametrize("d,ffn,relu_ffn,sizes,both", ONE_LAUNCH)
def test_ffn_products_in_one_launch(d, ffn, relu_ffn, sizes, both, form, ffn_options):
    """Both products in one launch against a launch each (which a given walk over the tiles asks for): the same bits, call after
    call and replayed from a graph with other rows in between."""
    ffn = relu_ffn if form == "relu" else ffn
    ffn_options()
    E, A, k = len(sizes), sum(sizes), 2
    A -= A % k
    sizes = [*sizes[:-1], sizes[-1] - sum(sizes) % k]
    gen = torch.Generator(device="cuda").manual_seed(81)
    bf = lambda *shape: torch.randn(shape, device="cuda", generator=gen).mul_(0.05).to(torch.bfloat16)
    W1, W3, W2 = bf(E, d, ffn), bf(E, d, ffn), bf(E, ffn, d)
    relu = form == "relu"
    packed = B.moe_pack_weights_relu(W1, W2) if relu else B.moe_pack_weights(W1, W3, W2)
    nseg = E + 2
    # expert 0 in two slots, one slot empty
    rows = [sizes[0] // 2, *sizes[1:], sizes[0] - sizes[0] // 2, 0]
    so, se = dev_i32(np.concatenate([[0], np.cumsum(rows)])), dev_i32([*range(E), 0, -1])
    of = torch.randperm(A, device="cuda", generator=gen).to(torch.int32)
    gate = torch.rand((A // k, k), device="cuda", generator=gen)
    xs = [bf(A // k if form in ("gather", "weights") else A, d) * 20 for _ in range(2)]
    ws = torch.zeros(B.moe_grouped_ffn_workspace_bytes(A, d, ffn, nseg, B.MOE_DTYPE_BF16), dtype=torch.uint8, device="cuda")
    y = torch.empty((A, d), dtype=torch.bfloat16, device="cuda")

    def call(x):
        if form in ("gather", "weights"):
            B.moe_grouped_ffn_gather(x, of, k, so, se, packed, E, ffn, workspace=ws, out=y, topk_w=gate if form == "weights" else None)
        else:
            B.moe_grouped_ffn(x, so, se, packed, E, ffn, workspace=ws, out=y, relu=relu)

    want = []
    for x in xs:
        ffn_options(group_n=4)
        y.fill_(-7)
        call(x)
        want.append(y.clone())
    ffn_options()
    for i in range(12):
        ws.fill_(255 if i % 3 == 0 else 0)
        y.fill_(-7)
        call(xs[i % 2])
        assert torch.equal(y, want[i % 2]), i
    x = xs[0].clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(x)
    for i in range(6):
        x.copy_(xs[i % 2])
        y.fill_(-7)
        graph.replay()
        assert torch.equal(y, want[i % 2]), i
    ref = torch.cat([(torch.relu(v @ W1[e].double()) if relu else torch.nn.functional.silu(v @ W1[e].double()) * (v @ W3[e].double()))
                     .to(torch.bfloat16).double() @ W2[e].double()
                     for e, v in zip([*range(E), 0], (xs[0] if form not in ("gather", "weights") else xs[0][of.long() // k])
                                     .double().split(rows[:-1]))])
    if form == "weights":
        ref *= gate.reshape(-1)[of.long()].double()[:, None]
    assert float((want[0].double() - ref).abs().max()) <= TOL["bf16"] * float(ref.abs().max())


def test_ffn_products_in_one_launch_on_two_streams(ffn_options):
    """Launches whose workgroups wait for each other's tiles, side by side on two streams: a tile belongs to a workgroup that
    runs, so either launch ends whatever part of it the other leaves room for."""
    ffn_options()
    d, ffn, E, sizes = 1024, 2048, 8, [700, 1, 0, 900, 513, 256, 1024, 702]
    A, nseg = sum(sizes), len(sizes)
    gen = torch.Generator(device="cuda").manual_seed(82)
    bf = lambda *shape: torch.randn(shape, device="cuda", generator=gen).mul_(0.05).to(torch.bfloat16)
    packed = B.moe_pack_weights(bf(E, d, ffn), bf(E, d, ffn), bf(E, ffn, d))
    so, se = dev_i32(np.concatenate([[0], np.cumsum(sizes)])), dev_i32([*range(E)])
    xs = [bf(A, d) * 20 for _ in range(2)]
    ws = [torch.zeros(B.moe_grouped_ffn_workspace_bytes(A, d, ffn, nseg, B.MOE_DTYPE_BF16), dtype=torch.uint8, device="cuda")
          for _ in range(2)]
    want = [B.moe_grouped_ffn(x, so, se, packed, E, ffn, workspace=w).clone() for x, w in zip(xs, ws)]
    ys = [[torch.empty((A, d), dtype=torch.bfloat16, device="cuda") for _ in range(8)] for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for i in range(8):
        for j, st in enumerate(streams):
            with torch.cuda.stream(st):
                B.moe_grouped_ffn(xs[j], so, se, packed, E, ffn, workspace=ws[j], out=ys[j][i])
    torch.cuda.synchronize()
    for j in range(2):
        for y in ys[j]:
            assert torch.equal(y, want[j]), j


@pytest.mark.parametrize("shift", [0, 16, 64, 112, 128])
def test_ffn_scratch_at_any_sixteen_bytes(shift, ffn_options):
    """The ABI asks 16 bytes of alignment of the scratch: hidden rows that share cache lines give the same bits."""
    ffn_options()
    d, ffn, E, sizes = 1024, 2048, 8, [700, 1, 0, 900, 513, 256, 1024, 702]
    A, nseg = sum(sizes), len(sizes)
    gen = torch.Generator(device="cuda").manual_seed(83)
    bf = lambda *shape: torch.randn(shape, device="cuda", generator=gen).mul_(0.05).to(torch.bfloat16)
    packed = B.moe_pack_weights(bf(E, d, ffn), bf(E, d, ffn), bf(E, ffn, d))
    so, se = dev_i32(np.concatenate([[0], np.cumsum(sizes)])), dev_i32([*range(E)])
    x, other = bf(A, d) * 20, bf(A, d) * 20
    n = B.moe_grouped_ffn_workspace_bytes(A, d, ffn, nseg, B.MOE_DTYPE_BF16)
    store = torch.zeros(n + 256, dtype=torch.uint8, device="cuda")
    at = -store.data_ptr() % 128 + shift
    want = B.moe_grouped_ffn(x, so, se, packed, E, ffn, workspace=store[at:at + n]).clone()
    ffn_options(group_n=4)   # a launch each
    assert torch.equal(B.moe_grouped_ffn(x, so, se, packed, E, ffn, workspace=store[at:at + n]), want)
    ffn_options()
    for _ in range(4):
        B.moe_grouped_ffn(other, so, se, packed, E, ffn, workspace=store[at:at + n])
        assert torch.equal(B.moe_grouped_ffn(x, so, se, packed, E, ffn, workspace=store[at:at + n]), want)
