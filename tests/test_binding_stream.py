"""The binding's current stream, on the CPU: by torch's raw handle where torch
has it, else by a stream object; a given stream as it is."""
import types

import pytest


@pytest.fixture
def binding(monkeypatch):
    import torch
    from paper_2110_11226_amd import _binding
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=11))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 100 + d, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    return _binding


def test_raw_handle_of_the_current_device(binding):
    assert binding._stream() == 103


@pytest.mark.parametrize("name", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_without_the_private_functions(binding, monkeypatch, name):
    import torch
    monkeypatch.delattr(torch._C, name)
    assert binding._stream() == 11


def test_before_torch_is_initialised(binding, monkeypatch):
    import torch
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    assert binding._stream() == 11


def test_a_given_stream(binding):
    assert binding._stream(types.SimpleNamespace(cuda_stream=5)) == 5
