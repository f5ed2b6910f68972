"""CPU checks of the pre-allocated runs: what a step hands to the library, seen by a stub in the library's place."""
import ctypes

import pytest
import torch

from paper_2401_08383_amd import binding as B
from paper_2401_08383_amd.pipeline import AffinityRun, MoELayerRun

LAYER_TENSORS = {  # attribute of the run -> field of the descriptor
    "x": "x", "w_gate": "w_gate", "w1": "w1", "w2": "w2", "forced_idx": "forced_idx", "expert_map": "expert_map", "topk_idx": "topk_idx",
    "topk_w": "topk_w", "x_sorted": "x_sorted", "src_of_sorted": "src_of_sorted", "sorted_of_src": "sorted_of_src",
    "expert_counts": "expert_counts", "expert_offsets": "expert_offsets", "y_sorted": "y_sorted", "out": "out",
    "ws_dispatch": "dispatch_workspace", "ws_ffn": "ffn_workspace"}


@pytest.fixture(autouse=True)
def _no_stream(monkeypatch):
    monkeypatch.setattr(B, "_stream", lambda: 0)


class LayerStub:
    """Records the descriptor of every moe_layer_forward call."""

    def __init__(self):
        self.seen = []

    def moe_layer_forward(self, address, stream):
        d = B.MoELayerDesc.from_address(address)
        self.seen.append({name: getattr(d, name) for name, _ in d._fields_})
        return 0


def _layer_run(fused):
    T, d, f, E, k = 5, 64, 128, 4, 2
    z = lambda *shape: torch.zeros(shape, dtype=torch.bfloat16)
    run = MoELayerRun(z(T, d), z(E, d), z(E, f, d), z(E, d, f), k, True, expert_map=torch.arange(E, dtype=torch.int32),
                      topk_idx=torch.zeros((T, k), dtype=torch.int32), fused=fused)
    run.lib = LayerStub()
    return run


def _expect(run):
    want = {}
    for attr, field in LAYER_TENSORS.items():
        t = getattr(run, attr)
        want[field] = None if t is None else t.data_ptr()
    want["dispatch_workspace_bytes"] = run.ws_dispatch.numel()
    want["ffn_workspace_bytes"] = run.ws_ffn.numel()
    return want


@pytest.mark.parametrize("how", ["data", "set_", "assign"])
@pytest.mark.parametrize("fused", [True, False])
def test_a_step_uses_the_storage_its_tensors_have_now(fused, how):
    """A tensor of the run whose storage was replaced in place between two steps: the next step gets the new address."""
    run = _layer_run(fused)
    run.step()
    kept = []
    for attr in LAYER_TENSORS:
        t = getattr(run, attr)
        if t is None:
            continue
        new = torch.zeros((t.numel() + 64,) if attr.startswith("ws_") else t.shape, dtype=t.dtype)
        kept.append(t.data)  # the old storage stays alive: its address is not given out again
        if how == "data":
            t.data = new
        elif how == "set_":
            t.set_(new)
        else:
            setattr(run, attr, new)
        run.step()
        got = run.lib.seen[-1]
        for field, value in _expect(run).items():
            assert got[field] == value, (attr, field)
        assert got[LAYER_TENSORS[attr]] == new.data_ptr()
    assert len(run.lib.seen) == 1 + len(kept)


def test_a_step_describes_the_assigned_values():
    run = _layer_run(True)
    run.step()
    run.renorm, run.act, run.forced_idx = 0, B.EXF_ACT_GELU_TANH, None
    run.step()
    got = run.lib.seen[-1]
    assert (got["renormalize"], got["act"], got["forced_idx"]) == (0, B.EXF_ACT_GELU_TANH, None)


def test_the_statistic_uses_the_storage_its_tensors_have_now():
    calls = []

    class Stub:
        def affinity_statistics(self, *args):
            calls.append(args)
            return 0

    run = AffinityRun(torch.zeros((3, 40), dtype=torch.int32), torch.zeros((3, 4), dtype=torch.int32), 4, 2)
    run.lib = Stub()
    run.step()
    for attr in ("trace", "placement", "counts", "loads", "cond_prob", "n_invalid", "local_per_pair", "ws_hist"):
        t = getattr(run, attr)
        old = t.data
        t.data = torch.zeros_like(t)
        run.step()
        assert t.data_ptr() != old.data_ptr()
        names = ("trace", "placement", None, None, None, None, "counts", "loads", "cond_prob", "n_invalid", "local_per_pair", "ws_hist")
        assert [calls[-1][i] for i, n in enumerate(names) if n] == [getattr(run, n).data_ptr() for n in names if n], attr


class CallsStub(LayerStub):
    """Records the entry points called, moe_layer_forward and the single ones."""

    def __getattr__(self, name):
        def call(*args):
            self.seen.append(name)
            return 0

        if name.startswith("__"):
            raise AttributeError(name)
        return call


@pytest.mark.parametrize("name", ["gate", "dispatch", "ffn", "combine"])
@pytest.mark.parametrize("where", ["subclass", "instance", "class"])
def test_a_step_goes_through_methods_that_were_replaced(monkeypatch, name, where):
    """A subclass's method or a hook around one of the four calls is part of the step, as long as it is there."""
    hooked = []
    original = getattr(MoELayerRun, name)

    def hook(self):
        hooked.append(name)
        original(self)

    run = _layer_run(False)
    run.lib = CallsStub()
    run.step()
    assert len(run.lib.seen) == 1 and isinstance(run.lib.seen[0], dict)  # one native call
    if where == "subclass":
        run.__class__ = type("Timed", (MoELayerRun,), {name: hook})
    elif where == "instance":
        setattr(run, name, lambda: hook(run))
    else:
        monkeypatch.setattr(MoELayerRun, name, hook)
    run.step()
    assert hooked == [name]
    assert run.lib.seen[1:] == ["moe_gate_topk", "moe_dispatch", "moe_expert_ffn", "moe_combine"]
    if where == "subclass":
        run.__class__ = MoELayerRun
    elif where == "instance":
        delattr(run, name)
    else:
        monkeypatch.undo()
        monkeypatch.setattr(B, "_stream", lambda: 0)
    run.step()
    assert hooked == [name] and isinstance(run.lib.seen[-1], dict) and len(run.lib.seen) == 6
