"""The handle of the current stream that the binding gives to the library, with and without torch's private lookup."""
import importlib.util
import types

import pytest
import torch

from paper_2603_06274_amd import binding as sb


def test_stream_without_the_private_lookup(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=4711))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    spec = importlib.util.spec_from_file_location("binding_again", sb.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    assert again._stream() == 4711


@pytest.mark.gpu
def test_stream_is_the_current_one(monkeypatch):
    stream = torch.cuda.Stream()
    for _ in range(2):
        assert sb._stream() == torch.cuda.current_stream().cuda_stream != stream.cuda_stream
        with torch.cuda.stream(stream):
            assert sb._stream() == stream.cuda_stream
        monkeypatch.setattr(sb, "_raw_stream", None)
