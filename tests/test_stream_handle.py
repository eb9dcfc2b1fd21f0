"""The stream handle the binding passes on: torch's current one by the raw call or, in a torch without
that (private) call, from the Stream object (no GPU needed)."""
from types import SimpleNamespace

import torch

from paper_1409_1510_amd import hisq

RAW = "_cuda_getCurrentRawStream"


def test_current_stream_with_and_without_the_raw_call(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=0x77))
    monkeypatch.setattr(torch._C, RAW, lambda device: 0x1000 + device, raising=False)
    assert hisq._stream_ptr(None).value == 0x1003
    monkeypatch.delattr(torch._C, RAW)
    assert hisq._stream_ptr(None).value == 0x77
