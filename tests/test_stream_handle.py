"""The handle of the stream that a call without one goes to: torch's own entry for it where there is one, the public
Stream object otherwise."""
import pytest
import torch

from paper_2602_22575_amd import binding


class _Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


@pytest.mark.parametrize("handle", [0, 0x7f00])
def test_current_stream_without_the_raw_entry(monkeypatch, handle):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: _Stream(handle))
    assert binding._stream_handle(None) == (handle or None)


@pytest.mark.parametrize("handle", [0, 0x7f00])
def test_current_stream_with_it(monkeypatch, handle):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: handle + device, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    assert binding._stream_handle(None) == (handle or None)


@pytest.mark.parametrize("handle", [0, 0x7f00])
def test_a_stream_that_is_given(handle):
    assert binding._stream_handle(_Stream(handle)) == (handle or None)
