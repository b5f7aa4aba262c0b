"""The handle of the current stream, with and without torch's shortcut to it."""
import types

import torch

import paper_2512_15187_amd as pid


def test_without_the_shortcut(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1230))
    assert pid._stream_ptr(None).value == 0x1230


def test_with_the_shortcut(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x4560 + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 1)
    assert pid._stream_ptr(None).value == 0x4561


def test_given_stream():
    assert pid._stream_ptr(types.SimpleNamespace(cuda_stream=0x7890)).value == 0x7890
