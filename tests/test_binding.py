"""The ctypes binding's own logic (no library call)."""

import types

import torch

from paper_2507_02754_amd import binding


def test_stream_without_the_raw_query(monkeypatch):
    """A torch without the raw stream query: the public Stream object's handle."""
    seen = []

    def current_stream(device):
        seen.append(device)
        return types.SimpleNamespace(cuda_stream=1234)

    monkeypatch.setattr(binding, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    device = torch.device("cuda", 3)
    assert binding._stream(device) == 1234 and seen == [device]
    monkeypatch.setattr(binding, "_raw_stream", lambda index: 10 + index)
    assert binding._stream(device) == 13 and len(seen) == 1
