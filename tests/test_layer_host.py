"""Which library calls a layer-step makes and in what order, with the calls recorded instead of made (no GPU)."""
import pytest
import torch

from paper_2506_05096_amd import binding as ab
from paper_2506_05096_amd import layer as al

N, H, D, K = 64, 2, 128, 20


@pytest.fixture
def calls(monkeypatch):
    made = []
    for name in ab.EXPORTS:
        if name in ("astraea_score", "astraea_select_topk", "astraea_kv_refresh", "astraea_scatter_update",
                    "astraea_lse_weight_update") or name.startswith("astraea_sparse_attn"):
            monkeypatch.setattr(ab, name, lambda *a, name=name, **kw: made.append(name[len("astraea_"):]))
    return made


def _inputs():
    rows = lambda: torch.zeros(N, H, D)
    return {"x_cur": torch.zeros(N, 64), "x_prev": torch.zeros(N, 64), "q": rows(), "k_cache": rows(), "v_cache": rows(),
            "k_new": rows(), "v_new": rows(), "out_cache": torch.zeros(N, H * D)}


def _layer(cls, fused=False):
    if issubclass(cls, al.StatefulLayer):
        return cls(N, H, D, 64, torch.float32, torch.ones(4), device="cpu", fused_update=fused)
    return cls(N, H, D, torch.float32, device="cpu", fused_update=fused)


HEAD = ["score", "select_topk", "kv_refresh"]
STATE = ["scatter_update", "lse_weight_update"]


def test_calls_of_a_step(calls):
    _layer(al.LayerStep).run(_inputs(), K)
    assert calls == HEAD + ["sparse_attn_scatter_fwd"]
    calls.clear()
    _layer(al.LayerStep, fused=True).run(_inputs(), K)
    assert calls == HEAD + ["sparse_attn_update_fwd"]
    calls.clear()
    _layer(al.StatefulLayer).run(_inputs(), K)
    assert calls == HEAD + ["sparse_attn_scatter_fwd"] + STATE
    calls.clear()
    _layer(al.StatefulLayer, fused=True).run(_inputs(), K)
    assert calls == HEAD + ["sparse_attn_update_fwd"] + STATE


# A step of a subclass, of an instance (a hook or a timer around it) or patched into the class is called, and in the order attention,
# state, scatter: a state step of one's own sees the cached outputs of the step before.
@pytest.mark.parametrize("cls", [al.LayerStep, al.StatefulLayer])
@pytest.mark.parametrize("name", ["step_attn", "step_state", "step_scatter"])
@pytest.mark.parametrize("where", ["subclass", "instance", "class"])
def test_replaced_steps_are_called(calls, monkeypatch, cls, name, where):
    if not hasattr(cls, name):
        pytest.skip("no such step")
    home = al.StatefulLayer if name == "step_state" else al.LayerStep
    own = getattr(home, name)

    def step(self, t, k, **kw):
        calls.append("own " + name)
        own(self, t, k, **kw)
    if where == "subclass":
        cls = type("Sub", (cls,), {name: step})
    elif where == "class":
        monkeypatch.setattr(home, name, step)
    layer = _layer(cls)
    if where == "instance":
        setattr(layer, name, lambda t, k, **kw: step(layer, t, k, **kw))
    layer.run(_inputs(), K)
    tail = {"step_attn": ["sparse_attn_fwd"], "step_state": STATE, "step_scatter": ["scatter_update"]}
    tail[name] = ["own " + name] + tail[name]
    stateful = issubclass(cls, al.StatefulLayer)
    assert calls == HEAD + tail["step_attn"] + (tail["step_state"] if stateful else []) + tail["step_scatter"]
