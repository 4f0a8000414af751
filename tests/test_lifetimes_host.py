"""What the Python objects keep alive, and which stream they name (no GPU)."""
import gc
import types
import weakref

import pytest
import torch

import paper_2605_14780_amd as hb


def test_graph_keeps_its_plan_and_fields(monkeypatch):
    """A replay reads the plan's tables, so a graph outlives neither its plan
    nor its fields, also where the caller drops them."""
    p = hb.Program(hb.Grid.cubed_sphere(4, 1))
    p.cs_add(4, 1, hb.CS_SYNC)
    plan = hb.Plan(p, host_only=True)
    fields = [type("Field", (), {})()]
    monkeypatch.setattr(hb, "_field", lambda plan, t: (hb.P(16), 1))
    monkeypatch.setattr(hb, "_stream", lambda stream: hb.P(16))
    monkeypatch.setattr(hb, "lib", lambda: types.SimpleNamespace(hbc_graph_create=lambda *a: hb.OK))
    graph = hb.ApplyGraph(plan, fields, 1)
    alive = [weakref.ref(plan), weakref.ref(fields[0])]
    del plan, fields
    gc.collect()
    assert all(r() is not None for r in alive)
    del graph
    gc.collect()
    assert all(r() is None for r in alive)


@pytest.mark.parametrize("name", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_torch_private_names(monkeypatch, name):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=48))
    for n in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.setattr(torch._C, n, lambda *a: 0, raising=False)
    monkeypatch.delattr(torch._C, name)
    assert hb._stream(None).value == 48
