"""A single step of MoELayer that a program has replaced is the one that ``step`` calls (no GPU needed)."""
import pytest
import torch

from paper_2506_07366_amd import binding as B
from paper_2506_07366_amd import workloads as wl
from paper_2506_07366_amd.layer import MoELayer

STEPS = ["route", "histogram", "plan", "permute", "ffn", "combine"]


@pytest.mark.parametrize("where", ["object", "class", "subclass"])
@pytest.mark.parametrize("replaced", STEPS)
def test_a_replaced_step_is_called(replaced, where, monkeypatch):
    cfg = wl.CONFIGS["mid_bf16"].replace(T=16, mode=wl.MODE_DISTRIBUTION)
    calls = []

    def spy(name):
        return lambda *a, **k: calls.append(name)

    cls = type("Sub", (MoELayer,), {replaced: spy(replaced)}) if where == "subclass" else MoELayer
    layer = cls(cfg, device="cpu")
    layer.packed = torch.empty(256, dtype=torch.uint8)     # (weights that nothing reads)
    layer._hp = layer._x = None                            # (what plan and permute leave to later steps)
    if where == "object":
        monkeypatch.setattr(layer, replaced, spy(replaced))
    elif where == "class":
        monkeypatch.setattr(MoELayer, replaced, spy(replaced))
    for n in STEPS:                                        # the library's own calls, which would need a GPU
        monkeypatch.setattr(B, {"plan": "moe_plan_duplicates", "ffn": "moe_grouped_ffn",
                                "route": "moe_route_topk"}.get(n, "moe_" + n), spy(n))
    logits, x = torch.zeros((cfg.T, cfg.E)), torch.zeros((cfg.T, cfg.d), dtype=torch.bfloat16)
    assert layer.step(logits, x, hist_pred=torch.ones(cfg.E, dtype=torch.int32)) is layer.out
    assert calls == STEPS


def test_a_layer_as_it_is_takes_the_one_call(monkeypatch):
    cfg = wl.CONFIGS["mid_bf16"].replace(T=16, mode=wl.MODE_NONE)
    layer = MoELayer(cfg, device="cpu")
    layer.packed = torch.empty(256, dtype=torch.uint8)
    calls = []
    monkeypatch.setattr(B, "moe_layer_step", lambda *a, **k: calls.append(k["x"]))
    x = torch.zeros((cfg.T, cfg.d), dtype=torch.bfloat16)
    layer.step(torch.zeros((cfg.T, cfg.E)), x)
    assert len(calls) == 1 and calls[0] is x
