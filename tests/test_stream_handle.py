"""The current stream's handle, with and without torch's private accessors."""
import types

import torch

import paper_2104_06311_amd as md


def test_public_property_where_torch_has_no_direct_accessor(monkeypatch):
    monkeypatch.setattr(md, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x7F0012345678))
    assert md._stream() == 0x7F0012345678


def test_direct_accessor(monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(md, "_raw_device", lambda: 3)
    monkeypatch.setattr(md, "_raw_stream", lambda dev: 0x1000 + dev)
    assert md._stream() == 0x1003
