"""The stream that calls are enqueued on: torch's current one, also with a torch that lacks the short way to its handle."""
import types

import pytest
import torch

from paper_2604_18655_amd import binding


@pytest.fixture
def fresh():
    binding._forget_device()
    yield
    binding._forget_device()


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_without_the_raw_handle(monkeypatch, fresh, missing):
    asked = []
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: asked.append(device) or types.SimpleNamespace(cuda_stream=4711))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.delattr(torch._C, missing, raising=False)
    assert binding._stream() == 4711
    assert asked[-1] in (None, 3)


@pytest.mark.gpu
def test_is_torchs_current_stream(gpu, fresh):
    side = torch.cuda.Stream()
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert binding._stream() == side.cuda_stream
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
