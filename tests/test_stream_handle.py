"""The stream handle the binding passes on: torch's raw query where torch has
it, a stream object's handle where it has not."""
import types

import pytest
import torch

from paper_2305_09163_amd import mfc


def test_given_stream():
    assert mfc._stream(types.SimpleNamespace(cuda_stream=4096)).value == 4096


def test_raw_query(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 4096 + device, raising=False)
    assert mfc._stream().value == 4099


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_without_the_raw_query(monkeypatch, missing):
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 4096 + device, raising=False)
    monkeypatch.delattr(torch._C, missing)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=8192))
    assert mfc._stream().value == 8192
