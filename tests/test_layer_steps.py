"""A forward whose steps are overridden calls them (no GPU: the library calls
are replaced by a record of their names)."""
import pytest
import torch

from paper_2205_01848_amd import MoELayer, rows_alloc_for
from paper_2205_01848_amd import binding as B

T, d, E, k, f = 8, 16, 4, 2, 32
CALLS = {"gate": "moe_gate_topk", "count": "moe_count", "capacity_static": "moe_update_capacity",
         "capacity_dynamic": "moe_update_capacity", "dispatch": "moe_dispatch",
         "ffn_fwd": "moe_expert_ffn_fwd", "combine": "moe_combine"}
SEPARATE = {"dynamic": ["moe_gate_topk", "moe_count", "moe_update_capacity", "moe_dispatch",
                        "moe_expert_ffn_fwd", "moe_combine"]}
SEPARATE["static"] = [c for c in SEPARATE["dynamic"] if c != "moe_count"]


@pytest.fixture
def calls(monkeypatch):
    seen = []
    for name in sorted(set(CALLS.values())) + ["moe_route", "moe_layer_fwd"]:
        monkeypatch.setattr(B, name, lambda *a, _n=name, **kw: seen.append(_n))
    return seen


def _forward(layer, kind):
    t = torch.zeros
    layer.forward(t(T, d), t(E, f, d), None, t(E, d, f), w_g=t(E, d), renorm=1,
                  capacity=(kind, 5, 4))


def _layer(cls=MoELayer):
    return cls(T, d, E, k, f, "relu", torch.float32, rows_alloc_for("dynamic", T, k, E, 5, 4),
               device="cpu")


@pytest.mark.parametrize("kind", ["static", "dynamic"])
def test_own_steps_are_one_call(calls, kind):
    _forward(_layer(), kind)
    assert calls == ["moe_layer_fwd"]


@pytest.mark.parametrize("kind", ["static", "dynamic"])
@pytest.mark.parametrize("how", ["subclass", "instance", "class"])
@pytest.mark.parametrize("step", sorted(CALLS))
def test_overridden_step_is_called(calls, monkeypatch, kind, how, step):
    own, hits = getattr(MoELayer, step), []

    def hook(self, *a, **kw):
        hits.append(step)
        return own(self, *a, **kw)

    cls = MoELayer
    if how == "subclass":
        cls = type("Hooked", (MoELayer,), {step: hook})
    elif how == "class":
        monkeypatch.setattr(MoELayer, step, hook)
    layer = _layer(cls)
    if how == "instance":
        setattr(layer, step, hook.__get__(layer))
    _forward(layer, kind)
    assert calls == SEPARATE[kind]
    assert hits == ([step] if CALLS[step] in calls and step != {"static": "capacity_dynamic",
                                                                "dynamic": "capacity_static"}[kind]
                    else [])
