"""The stream a call goes to (no GPU): the given one, else torch's current one,
with or without torch's function that returns the bare handle."""
import types

import pytest

from paper_2208_12795_amd import etpic as E


def stream(handle):
    return types.SimpleNamespace(cuda_stream=handle)


@pytest.mark.parametrize("raw", [None, lambda device: 77 if device == 3 else -1])
def test_stream_handle(monkeypatch, raw):
    cuda = types.SimpleNamespace(current_stream=lambda: stream(77), current_device=lambda: 3)
    monkeypatch.setattr(E, "_torch", types.SimpleNamespace(cuda=cuda))
    monkeypatch.setattr(E, "_raw_stream", raw)
    assert E._stream(None) == 77
    assert E._stream(stream(5)) == 5


def test_torch_without_the_bare_handle(monkeypatch):
    import torch
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(E, "_torch", None)
    monkeypatch.setattr(E, "_raw_stream", "unset")
    E._load_torch()
    assert E._raw_stream is None
