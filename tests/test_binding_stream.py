"""The binding asks torch for the current stream's handle by two private names; without them it falls back to the public
call.  Host only: torch's side is replaced."""
import importlib.util
import types

import pytest
import torch

import paper_2105_14088_amd.binding as binding

PRIVATE = ("_cuda_getDevice", "_cuda_getCurrentRawStream")


@pytest.mark.parametrize("missing", [PRIVATE, PRIVATE[:1], PRIVATE[1:]])
def test_import_and_current_stream_without_the_private_names(monkeypatch, missing):
    for name in missing:
        monkeypatch.delattr(torch._C, name, raising=False)
    spec = importlib.util.spec_from_file_location("binding_without_private_names", binding.__file__)
    fresh = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(fresh)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x5EED))
    assert fresh._stream(None) == 0x5EED
    assert fresh._stream(types.SimpleNamespace(cuda_stream=0x1234)) == 0x1234


def test_private_names_give_the_current_device_s_stream(monkeypatch):
    monkeypatch.setattr(binding, "_current_device", lambda: 3)
    monkeypatch.setattr(binding, "_current_raw_stream", lambda device: 100 + device)
    assert binding._stream(None) == 103
