"""What a user of the library runs, as a set of timed cases.

A case is one pass of ``MoELayer`` (route, histogram, duplication plan, permute, grouped FFN,
combine) over one batch that is resident in device memory, on a shape of
``paper_2506_07366_amd.workloads.CONFIGS`` at some number of tokens.  Fields of a case:

  shape   name in CONFIGS: widths, experts, ranks, slots, data type, form of the FFN
  tokens  tokens of the batch
  mode    plan: 0 home placement, 1 Distribution-Only, 2 Token-to-Expert
  path    "copied"  six calls, the permuted rows are materialised (the default of MoELayer)
          "gather"  the first product gathers the token rows itself
          "weights" and the second product applies the gate weights
          "graph"   the copied path recorded once with MoELayer.capture and replayed
          "stream"  the copied path inside the loop of the Distribution-Only predictor: the
                    plan takes the running estimate, the batch's histogram goes into it, and
                    the rows that cross ranks are counted
  alpha   Dirichlet concentration of the expert popularity (shapes with Zipf popularity keep it)

Inputs come from the case's seed alone and are drawn on the device: router logits N(0, 1) +
log popularity, activations N(0, 1), weights N(0, 0.02), predicted histograms and predicted ids
with the noise the shape's configuration names.
"""
import numpy as np
import torch

from paper_2506_07366_amd import binding as B
from paper_2506_07366_amd import workloads as wl
from paper_2506_07366_amd.layer import MoELayer, torch_dtype

# tokens each shape is used at, and the paths of its form of the FFN
RANGES = {
    "cfg1_tiny_f32": (16, 2048, ("copied", "gather", "weights", "graph")),
    "mid_bf16": (16, 4096, ("copied", "gather", "weights", "graph", "stream")),
    "cfg2_mixtral_dist": (1, 8192, ("copied", "gather", "weights", "graph", "stream")),
    "cfg4_finegrained": (16, 16384, ("copied", "gather", "weights", "stream")),
    "cfg5_decode_m1": (1, 32768, ("copied", "gather", "weights", "graph", "stream")),
    "cfg6_switch_relu": (16, 16384, ("copied", "graph")),
    "cfg7_llama_moe": (16, 8192, ("copied", "gather", "weights")),
}


def listed():
    c = lambda name, shape, tokens, mode, path, alpha=0.5: dict(name=name, shape=shape, tokens=tokens, mode=mode,
                                                                path=path, alpha=alpha)
    return [
        # the small fp32 layer that results are checked on: launches and host time
        c("tiny_f32", "cfg1_tiny_f32", 256, 1, "copied"),
        # one token of one sequence through a layer of many small experts: pure latency
        c("one_token", "cfg5_decode_m1", 1, 1, "weights", 1.0),
        # a small serving batch on few large experts, replayed as a graph the way a server would
        c("mixtral_decode_graph", "cfg2_mixtral_dist", 16, 1, "graph"),
        # a decode batch over many small experts with duplication: weights stream once per step
        c("decode_128", "cfg5_decode_m1", 128, 1, "copied", 1.0),
        # decode and short prompts mixed in one batch, ragged, with token-level predictions
        c("mixed_batch_777", "cfg5_decode_m1", 777, 2, "gather", 0.1),
        # a short prompt on few large experts, odd length
        c("mixtral_prompt_1001", "cfg2_mixtral_dist", 1001, 2, "copied"),
        # batches of a stream with the running predictor and the accounting of crossing rows
        c("stream_2048", "cfg4_finegrained", 2048, 1, "stream"),
        # prefill on few large experts: the benchmark's workload
        c("mixtral_prefill", "cfg2_mixtral_dist", 4096, 1, "copied"),
        # prefill on fine-grained experts with Zipf popularity
        c("finegrained_prefill", "cfg4_finegrained", 16384, 1, "copied"),
        # ReLU experts, top-1, narrow model
        c("switch_relu", "cfg6_switch_relu", 16384, 1, "copied"),
        # hidden width that is no multiple of the tile, odd number of tokens, no prediction
        c("llama_moe_8191", "cfg7_llama_moe", 8191, 0, "weights"),
        # the largest batch: long prefill over many small experts
        c("prefill_32768", "cfg5_decode_m1", 32768, 1, "copied", 1.0),
    ]


def draw(rng):
    shape = rng.choice(sorted(RANGES))
    lo, hi, paths = RANGES[shape]
    tokens = min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))
    path = rng.choice(paths)
    return dict(shape=shape, tokens=tokens, mode=1 if path == "stream" else rng.choice((0, 1, 2)), path=path,
                alpha=rng.choice((0.1, 0.5, 1.0, 10.0)))


def _config(case, seed):
    return wl.CONFIGS[case["shape"]].replace(name=case["shape"], T=case["tokens"], mode=case["mode"],
                                             alpha=case["alpha"], seed=seed)


def _weights(cfg, gen):
    dt = torch_dtype(cfg)

    def one(*shape):
        w = torch.empty(shape, dtype=dt, device="cuda")
        return w.normal_(0.0, 0.02, generator=gen)

    W1 = one(cfg.E, cfg.d, cfg.ffn)
    W3 = None if cfg.act == "relu" else one(cfg.E, cfg.d, cfg.ffn)
    return W1, W3, one(cfg.E, cfg.ffn, cfg.d)


def prepare(case, seed):
    cfg = _config(case, seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    path = case["path"]
    layer = MoELayer(cfg, fused_gather=path == "gather", fused_weights=path == "weights")
    layer.set_weights(*_weights(cfg, gen))
    bias = torch.from_numpy(np.log(wl.expert_popularity(cfg)).astype(np.float32)).cuda()
    logits = torch.randn((cfg.T, cfg.E), device="cuda", generator=gen) + bias
    x = torch.randn((cfg.T, cfg.d), device="cuda", generator=gen).to(torch_dtype(cfg))
    true_idx = torch.topk(logits, cfg.k, dim=1).indices
    true_hist = torch.bincount(true_idx.reshape(-1), minlength=cfg.E)
    state = dict(cfg=cfg, layer=layer, path=path, logits=logits, x=x, hist_pred=None, pred_idx=None)
    if path == "stream":
        # the predictor has seen an earlier batch of the same popularity
        seen = torch.randn((cfg.T, cfg.E), device="cuda", generator=gen) + bias
        seen_idx = torch.topk(seen, cfg.k, dim=1).indices.reshape(-1)
        state["counts"] = torch.bincount(seen_idx, minlength=cfg.E).to(torch.int64)
        state["hist_pred"] = torch.zeros(cfg.E, dtype=torch.int32, device="cuda")
    elif cfg.mode == wl.MODE_DISTRIBUTION:
        state["hist_pred"] = torch.from_numpy(wl.gen_pred_hist(cfg, true_hist.cpu().numpy())).cuda()
    elif cfg.mode == wl.MODE_TOKEN:
        # a token's row is predicted right with probability acc, else k distinct uniform ids
        keep = torch.rand((cfg.T, 1), device="cuda", generator=gen) < cfg.acc
        uniform = torch.rand((cfg.T, cfg.E), device="cuda", generator=gen).topk(cfg.k, dim=1).indices
        state["pred_idx"] = torch.where(keep, true_idx, uniform).to(torch.int32).contiguous()
    if path == "graph":
        state["graph"] = layer.capture(logits, x, hist_pred=state["hist_pred"], pred_idx=state["pred_idx"])
    return state


def _outputs(layer):
    p = layer.perm
    return dict(out=layer.out, topk_idx=layer.topk_idx, topk_w=layer.topk_w, hist=layer.hist,
                slot_expert=layer.slot_expert, slot_quota=layer.slot_quota, seg_offsets=p["seg_offsets"],
                row_of_assign=p["row_of_assign"], assign_of_row=p["assign_of_row"], rank_load=p["rank_load"])


def run(state):
    layer, cfg = state["layer"], state["cfg"]
    if state["path"] == "graph":
        state["graph"].replay()
        return _outputs(layer)
    if state["path"] == "stream":
        B.moe_predictor_predict(state["counts"], cfg.A, out=state["hist_pred"])
        layer.step(state["logits"], state["x"], hist_pred=state["hist_pred"])
        B.moe_predictor_update(layer.hist, state["counts"])
        dispatch, combine = B.moe_comm_matrix(cfg.mode, layer.topk_idx, None, layer.perm["row_of_assign"],
                                              layer.perm["seg_offsets"], cfg.G, cfg.S)
        return dict(_outputs(layer), counts=state["counts"], hist_pred=state["hist_pred"], dispatch=dispatch,
                    combine=combine)
    layer.step(state["logits"], state["x"], hist_pred=state["hist_pred"], pred_idx=state["pred_idx"])
    return _outputs(layer)


def _experts_with_rows(cfg):
    """Experts that a batch touches, averaged over a few popularities of the shape's kind."""
    tokens = min(cfg.T, 1024)
    n = []
    for seed in range(4):
        c = cfg.replace(T=tokens, seed=1000 + seed)
        idx = np.argpartition(-wl.gen_logits(c), cfg.k - 1, axis=1)[:, :cfg.k]
        n.append(np.unique(idx).size)
    return float(np.mean(n))


def work(case):
    cfg = _config(case, 0)
    size = 4 if cfg.dtype == "f32" else 2
    matrices = 2 if cfg.act == "relu" else 3
    weights = _experts_with_rows(cfg) * matrices * cfg.d * cfg.ffn * size
    rows = 2 * cfg.T * cfg.d * size               # x in, out out
    if case["path"] not in ("gather", "weights"):
        rows += cfg.A * cfg.d * size              # x_perm is an output of this path
    index = 4 * (cfg.T * cfg.E + 4 * cfg.A)       # logits in; ids, weights and both permutations out
    return {"bytes": weights + rows + index, "flops": 2.0 * matrices * cfg.A * cfg.d * cfg.ffn}


def tolerance(case):
    # fp32: sums of up to a few thousand products; bf16: hidden activation, expert result and
    # output are each rounded to 8 bits.  About four times what the path shows against the same
    # computation in 64 bits.
    if wl.CONFIGS[case["shape"]].dtype == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 1e-2, "max": 5e-2}
