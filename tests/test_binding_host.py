"""CPU-only: what the binding itself does between torch and the library."""
import types

import torch

from paper_2301_08739_amd import binding


def test_stream_without_the_short_way(monkeypatch):
    """The number of the current stream comes from a Stream object where this torch has no function for it."""
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4711))
    assert binding._stream() == 4711
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    assert binding._stream() == 103
