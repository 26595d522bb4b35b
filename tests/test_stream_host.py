"""The stream handle that the binding passes on, with and without torch's
private accessors."""
import types

import pytest
import torch

import paper_1711_07793_amd as rb


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_private_accessors(monkeypatch, missing):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.setattr(torch._C, name, lambda *args: 77, raising=False)
    assert rb._stream(None) == 77
    monkeypatch.delattr(torch._C, missing)
    assert rb._stream(None) == 1234


def test_given_streams():
    assert rb._stream(types.SimpleNamespace(cuda_stream=5)) == 5
    assert rb._stream(6) == 6
