"""The binding's stream handle on a torch that lacks the raw-stream function of its C module."""
from types import SimpleNamespace

import torch

import paper_2607_12696_amd as moe


def test_stream_without_the_raw_stream_function(monkeypatch):
    monkeypatch.setattr(moe, "_raw_stream", None, raising=False)
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: SimpleNamespace(cuda_stream=4096 + device))
    assert moe._stream(SimpleNamespace(get_device=lambda: 3)) == 4099
