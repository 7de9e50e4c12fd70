"""Host side of the binding (no GPU): the stream handle and the device that a
call asks torch for, with and without torch's private accessors."""
import contextlib
import importlib.util
import types

import pytest
import torch

from paper_1706_03292_amd import api


def _load(monkeypatch, private):
    """A second copy of the binding, in a torch that has the private accessors
    (here: stand-ins) or lacks them."""
    for name, value in (("_cuda_getCurrentRawStream", lambda i: 700 + i), ("_cuda_getDevice", lambda: 1)):
        if private:
            monkeypatch.setattr(torch._C, name, value, raising=False)
        else:
            monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d: types.SimpleNamespace(cuda_stream=700 + (d.index or 0)))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 1)
    monkeypatch.setattr(torch.cuda, "device", lambda d: contextlib.closing(types.SimpleNamespace(close=lambda: None)))
    spec = importlib.util.spec_from_file_location(api.__name__, api.__file__)
    copy = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(copy)
    return copy


@pytest.mark.parametrize("private", [True, False])
def test_binding_finds_stream_and_device_without_torchs_private_accessors(monkeypatch, private):
    copy = _load(monkeypatch, private)
    for index in (0, 1):
        assert copy._stream_handle(None, torch.device("cuda", index)) == 700 + index
    assert copy._stream_handle(None, torch.device("cuda")) == 700
    assert copy._stream_handle(types.SimpleNamespace(cuda_stream=5), torch.device("cuda", 0)) == 5
    assert copy._stream_handle(9, torch.device("cuda", 0)) == 9
    assert copy._on(torch.device("cuda", 1)) is copy._SAME_DEVICE
    for other in (torch.device("cuda", 0), torch.device("cuda")):
        assert isinstance(copy._on(other), contextlib.closing)
