"""The stream handle that the Python entry points hand to the library: the current
stream of the current device, from torch's raw handle where this torch has it and
from the public call where it does not."""
import types

import pytest
import torch

from paper_2609_36757_amd import fastvr


def test_given_stream_is_used():
    assert fastvr._stream_handle(types.SimpleNamespace(cuda_stream=77)) == 77


def test_raw_handle_of_the_current_device(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 1000 + d, raising=False)
    assert fastvr._stream_handle(None) == 1003


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_public_call_where_the_raw_handle_is_missing(monkeypatch, missing):
    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=55))
    assert fastvr._stream_handle(None) == 55


@pytest.mark.gpu
def test_handle_follows_the_current_stream():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("\n[gpu case] stream handle", flush=True)
    assert fastvr._stream_handle(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(torch.cuda.Stream()) as _:
        assert fastvr._stream_handle(None) == torch.cuda.current_stream().cuda_stream != 0
