"""The stream of a call: torch's raw handle where it has that function, else the Stream object's."""
import types

import pytest
import torch

from paper_1402_4986_amd import api


@pytest.mark.parametrize("raw", [True, False])
@pytest.mark.parametrize("index", [0, None])
def test_stream_handle(monkeypatch, raw, index):
    if raw:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda i: 100 + i, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: types.SimpleNamespace(cuda_stream=7))
    device = types.SimpleNamespace(index=index)
    assert api._stream_handle(device) == (100 if raw and index == 0 else 7)
