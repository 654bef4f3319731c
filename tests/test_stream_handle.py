"""The caller's current stream reaches the library also under a torch that lacks
the functions behind the raw handle (CPU only)."""
import pytest
import torch

from paper_2606_12688_amd import attn


@pytest.mark.parametrize("missing", [None, "_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream(monkeypatch, missing):
    class Stream:
        cuda_stream = 4242

    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 1000 + d, raising=False)
    if missing:
        monkeypatch.delattr(torch._C, missing)
    assert attn._stream_handle(None) == (1003 if missing is None else 4242)
    assert attn._stream_handle(Stream) == 4242 and attn._stream_handle(7) == 7
