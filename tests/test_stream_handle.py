"""The stream that a call is handed: the current one, by torch's raw handle or, with a torch that has no such thing, out of its Stream object."""
import importlib.util

import pytest
import torch

from paper_2511_11346_amd import binding


def without_raw_handle(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    spec = importlib.util.spec_from_file_location("binding_without_raw_handle", binding.__file__)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


def test_a_torch_without_the_raw_handle(monkeypatch):
    module = without_raw_handle(monkeypatch)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: type("Stream", (), {"cuda_stream": 4096 + device}))
    assert module._raw_stream(3) == 4099


@pytest.mark.gpu
def test_both_name_the_current_stream(monkeypatch):
    module = without_raw_handle(monkeypatch)
    monkeypatch.undo()
    for stream in (torch.cuda.default_stream(0), torch.cuda.Stream(0)):
        with torch.cuda.stream(stream):
            assert binding._raw_stream(0) == module._raw_stream(0) == stream.cuda_stream
