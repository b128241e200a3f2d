"""The stream a call is enqueued on is torch's current one, also with a torch
that lacks the private function the binding prefers."""
import importlib.util
import types

import pytest
import torch

from paper_2506_15050_amd import binding


def test_stream_without_private_torch_names(monkeypatch):
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=4096))
    spec = importlib.util.spec_from_file_location("binding_elsewhere", binding.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    assert again._stream() == 4096


@pytest.mark.gpu
def test_stream_is_the_current_one():
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert binding._stream() == side.cuda_stream
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
