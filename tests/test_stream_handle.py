"""The current stream's handle on a torch that does not give it directly."""
import types

import pytest

torch = pytest.importorskip("torch")

import paper_1705_09776_amd as cd  # noqa: E402


def test_handle_without_the_direct_call(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1230))
    assert cd._stream(None) == 0x1230


def test_handle_with_the_direct_call(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x4560 + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert cd._stream(None) == 0x4563
    assert cd._stream(7) == 7 and cd._stream(types.SimpleNamespace(cuda_stream=9)) == 9
