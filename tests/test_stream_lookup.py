"""The current stream's handle without torch's raw lookups (underscore names that
a torch may lack) and without an initialised device: the public way."""
import pytest
import torch

from paper_2606_20537_amd import _native as N


class Stream:
    cuda_stream = 77


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_torch_without_raw_lookups(monkeypatch, missing):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(N, "_raw", None)
    assert N._stream(None) == 77 and N._stream(None) == 77


@pytest.mark.parametrize("initialised", [False, True])
def test_raw_lookups_only_when_initialised(monkeypatch, initialised):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: initialised)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 1000 + device, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(N, "_raw", None)
    assert N._stream(None) == (1003 if initialised else 77)
    assert N._stream(5) == 5 and N._stream(Stream) == 77
