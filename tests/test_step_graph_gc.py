"""Capturing a step graph keeps Python's garbage collector out of the capture
(an engine or graph in a reference cycle would be destroyed inside it), also
while another thread's capture ends, and leaves the collector as it was."""
import contextlib
import gc
import threading
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


@pytest.mark.parametrize("enabled", [True, False])
def test_overlapping_captures_of_two_threads(enabled):
    entered, left = threading.Event(), threading.Event()
    was = gc.isenabled()
    (gc.enable if enabled else gc.disable)()

    def first():
        with sdrl.no_collection():
            entered.set()
            assert second_in.wait(20)
        left.set()

    second_in = threading.Event()
    t = threading.Thread(target=first)
    try:
        t.start()
        assert entered.wait(20)
        with sdrl.no_collection():
            second_in.set()
            assert left.wait(20)
            assert not gc.isenabled()                # the first capture has ended, this one has not
        assert gc.isenabled() == enabled
    finally:
        t.join()
        (gc.enable if was else gc.disable)()
