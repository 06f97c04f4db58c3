"""The stream handle that a call without a stream argument gets, where torch lacks the undocumented function for it (no GPU
involved: torch's side is stood in for)."""
import types

import torch

from paper_2010_00704_amd import binding as B


def test_current_stream_without_the_raw_handle(monkeypatch):
    monkeypatch.setattr(B, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    assert B._stream(None) == 1234


def test_raw_handle_is_of_the_current_device(monkeypatch):
    monkeypatch.setattr(B, "_raw_stream", lambda device: 100 + device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert B._stream(None) == 103
    assert B._stream(7) == 7
    assert B._stream(types.SimpleNamespace(cuda_stream=9)) == 9
