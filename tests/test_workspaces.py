"""The binding's workspaces: what a captured graph may hold stays allocated, and a
workspace made during a capture serves that capture alone.  (On the CPU: the
stream's handle and its capture are given.)"""
import gc
import weakref

import pytest

from paper_2310_07177_amd import binding


@pytest.fixture
def stream(monkeypatch):
    import torch
    state = {"handle": 7, "capture": 0}
    monkeypatch.setattr(binding, "_stream_handle", lambda device: state["handle"])
    monkeypatch.setattr(binding, "_capture_id", lambda handle: state["capture"], raising=False)
    for name in ("_workspaces", "_captured"):
        monkeypatch.setattr(binding, name, {}, raising=False)
    monkeypatch.setattr(binding, "_superseded", [], raising=False)
    state["get"] = lambda nbytes, kind="verify": binding.workspace(kind, nbytes, torch.device("cpu"))
    return state


def test_superseded_workspaces_stay_allocated(stream):
    refs, used = [], 0
    for nbytes in (300, 5000, 5001, 20000, 1000, 70000):
        refs.append(weakref.ref(stream["get"](nbytes)))
        assert refs[-1]().numel() >= nbytes and int(refs[-1]().sum()) == 0
    gc.collect()
    assert all(r() is not None for r in refs)
    assert refs[1]() is not refs[3]() and refs[4]() is refs[3]()
    # together smaller than the one in use
    now = stream["get"](70000)
    kept = {id(r()): r().numel() for r in refs if r() is not now}
    assert 0 < sum(kept.values()) < now.numel()


def test_workspace_of_a_capture(stream):
    stream["capture"] = 3
    first = stream["get"](1000)
    assert stream["get"](900) is first  # the same capture
    assert stream["get"](900, "distill") is not first
    stream["capture"] = 4
    assert stream["get"](900) is not first  # another graph's
    stream["capture"] = 0
    eager = stream["get"](900)
    assert eager is not first and stream["get"](1000) is eager
    stream["capture"] = 5
    assert stream["get"](1000) is eager  # made outside: zeroed, and every capture's
    stream["handle"] = 8
    assert stream["get"](1000) is not eager
