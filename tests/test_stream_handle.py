"""The handle of torch's current stream, with and without torch's private shortcut (CPU: torch's
functions are stood in for)."""
from __future__ import annotations

import os
import subprocess
import sys
from types import SimpleNamespace

import torch

from paper_2607_22648_amd import ptstore as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_current_stream_without_the_private_function(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(P, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=0x51))
    assert P._stream(None) == 0x51


def test_import_without_the_private_function():
    """The package imports where torch lacks it, and finds it missing."""
    code = ("import torch\n"
            "if hasattr(torch._C, '_cuda_getCurrentRawStream'): del torch._C._cuda_getCurrentRawStream\n"
            "from paper_2607_22648_amd import ptstore\n"
            "assert ptstore._raw_stream is None\n")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT)


def test_current_stream_by_the_private_function(monkeypatch):
    monkeypatch.setattr(P, "_raw_stream", lambda device: 0x70 + device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert P._stream(None) == 0x73
    assert P._stream(0x99) == 0x99  # a handle that the caller gives
