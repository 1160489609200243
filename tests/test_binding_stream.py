"""The stream that a call without one is issued on: the caller's, torch's current one by its
raw handle, or by the public call where torch has no such lookup."""
import torch

import paper_2505_22913_amd as mf


class _Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


def test_stream_handle(monkeypatch):
    assert mf._stream(_Stream(7)) == 7
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: _Stream(9))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
    assert mf._stream(None) == 103
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert mf._stream(None) == 9
