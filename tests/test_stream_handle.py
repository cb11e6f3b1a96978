"""The handle that a call passes on when no stream is given (no GPU: torch's functions are stand-ins)."""
import types

import torch

from paper_2605_07330_amd import srs


def test_without_the_raw_handle_function(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(srs, "_raw_stream", None, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1230))
    assert srs._stream_ptr(None) == 0x1230
    assert srs._stream_ptr(types.SimpleNamespace(cuda_stream=0x4560)) == 0x4560


def test_with_the_raw_handle_function(monkeypatch):
    monkeypatch.setattr(srs, "_raw_stream", lambda device: 0x1000 + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert srs._stream_ptr(None) == 0x1003
