"""The handle of torch's current stream, with and without torch's private shortcut (CPU: torch's
functions are stood in for)."""
from __future__ import annotations

from types import SimpleNamespace

import torch

from paper_2607_22648_amd import ptstore as P


def test_current_stream_without_the_private_function(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=0x51))
    assert P._stream(None) == 0x51


def test_current_stream_by_the_private_function(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x70 + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert P._stream(None) == 0x73
    assert P._stream(0x99) == 0x99  # a handle that the caller gives
