"""The stream a call without one goes to: the current one, by torch's handle function or, where a version of torch has none, by its public
Stream object."""
import types

import torch

from paper_2508_15706_amd import binding


def test_current_stream(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x70))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x50 + device, raising=False)
    assert binding._stream_ptr(None) == 0x53
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert binding._stream_ptr(None) == 0x70
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0))
    assert binding._stream_ptr(None) is None and binding._stream_ptr(0x90) == 0x90
