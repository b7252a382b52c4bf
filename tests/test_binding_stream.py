"""The stream that a call without one takes (CPU only): the current stream of
the current device, by torch's own lookup where it has one and by its public
interface where not."""
import types

import torch

import paper_2602_02071_amd as baps


def _as_initialised(monkeypatch, handle):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=handle))


def test_handle_lookup(monkeypatch):
    _as_initialised(monkeypatch, 7)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 2, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 100 + dev, raising=False)
    assert baps._stream(None) == 102


def test_without_the_handle_lookup(monkeypatch):
    _as_initialised(monkeypatch, 7)
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert baps._stream(None) == 7
    monkeypatch.delattr(torch._C, "_cuda_getDevice", raising=False)
    assert baps._stream(None) == 7


def test_given_streams():
    assert baps._stream(5) == 5
    assert baps._stream(types.SimpleNamespace(cuda_stream=9)) == 9
