"""The binding's stream handle: the given stream's, else the current one's, with and without torch's raw
handle."""
import types

import torch

from paper_2010_11540_amd import scpic


def test_stream_handle(monkeypatch):
    given = types.SimpleNamespace(cuda_stream=7)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=42))
    monkeypatch.setattr(scpic, "_raw_stream", lambda device: 100 + device)
    assert scpic._stream_ptr(given) == 7
    assert scpic._stream_ptr(None) == 103
    monkeypatch.setattr(scpic, "_raw_stream", None)
    assert scpic._stream_ptr(given) == 7
    assert scpic._stream_ptr(None) == 42
