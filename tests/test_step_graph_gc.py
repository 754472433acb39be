"""Capturing a step graph keeps Python's garbage collector out of the capture
(an engine or graph in a reference cycle would be destroyed inside it), and
leaves the collector as it was."""
import contextlib
import gc
import types

import pytest
import torch

from paper_2606_18967_amd import sdrl


@pytest.mark.parametrize("enabled", [True, False])
@pytest.mark.parametrize("fails", [False, True])
def test_no_collection_inside_the_capture(monkeypatch, enabled, fails):
    seen = []

    def step(*a):
        seen.append(gc.isenabled())
        if fails:
            raise RuntimeError("capture")

    stream = types.SimpleNamespace(wait_stream=lambda s: None)
    monkeypatch.setattr(sdrl, "sd_step", step)
    monkeypatch.setattr(torch.cuda, "CUDAGraph", lambda: None)
    monkeypatch.setattr(torch.cuda, "Stream", lambda device=None: stream)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: stream)
    monkeypatch.setattr(torch.cuda, "graph", lambda g, stream=None: contextlib.nullcontext())
    tok = torch.zeros(1, dtype=torch.int32)
    was = gc.isenabled()
    (gc.enable if enabled else gc.disable)()
    try:
        with pytest.raises(RuntimeError) if fails else contextlib.nullcontext():
            sdrl.StepGraph(types.SimpleNamespace(device=None), types.SimpleNamespace(next_tok=tok), tok, tok.clone(), 1.0,
                           0, 0)
        assert seen == [False] and gc.isenabled() == enabled
    finally:
        (gc.enable if was else gc.disable)()
