"""Which stream a call of the binding goes to: the one that is passed, else the current one, by its raw handle where torch
has the function and through the stream object where it does not."""
import types

import torch

from paper_2406_11430_amd import binding


def test_stream_that_is_passed():
    assert binding._stream(types.SimpleNamespace(cuda_stream=1234)) == 1234


def test_current_stream_by_raw_handle(monkeypatch):
    monkeypatch.setattr(binding, "_device_index", lambda: 3)
    monkeypatch.setattr(binding, "_raw_stream_of", lambda device: 100 + device)
    assert binding._stream(None) == 103


def test_current_stream_without_the_private_functions(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(binding, "_raw_stream_of", None)
    assert binding._stream(None) == 77
