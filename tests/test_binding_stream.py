"""The current stream's handle in a torch build that lacks the functions the
binding reads it with (no GPU: torch's stream object is a stand-in)."""
import types

import pytest
import torch

import paper_1012_2270_amd as rg


@pytest.mark.parametrize("lacks", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_without_private_functions(monkeypatch, lacks):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    monkeypatch.delattr(torch._C, lacks, raising=False)
    monkeypatch.setattr(rg, "_current_stream", None, raising=False)
    assert rg._stream() == 1234
    assert rg._astream(types.SimpleNamespace()) == 1234
    assert rg._stream(types.SimpleNamespace(cuda_stream=7)) == 7
