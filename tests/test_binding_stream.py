"""The stream handle that the binding passes: torch's own shortcut where this torch has it, the public interface where not."""
import types

import torch

from paper_2512_22804_amd import binding as B


def test_shortcut(monkeypatch):
    monkeypatch.setattr(B, "_raw_stream", lambda device: 1000 + device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert B._stream() == 1003


def test_public_interface(monkeypatch):
    monkeypatch.setattr(B, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert B._stream() == 77
