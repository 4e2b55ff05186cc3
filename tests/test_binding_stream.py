"""The current stream's address where torch has no lookup without a Stream object (host-only)."""
import importlib

import torch

from paper_2404_19124_amd import binding as B


def test_current_stream_without_the_raw_lookup(monkeypatch):
    class Stream:
        cuda_stream = 4711

    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.delattr(torch._C, "_cuda_getDevice", raising=False)
    binding = importlib.reload(B)   # (the names are looked up once)
    try:
        assert binding._stream_ptr(None) == 4711
    finally:
        monkeypatch.undo()
        importlib.reload(B)
