"""The stream a call gets when none is named: the current device's current stream, also on a torch without the private calls that
the binding takes it from where they exist."""
import pytest

from paper_2603_06199_amd import binding as B

torch = pytest.importorskip("torch")


class Stream:
    def __init__(self, raw):
        self.cuda_stream = raw


@pytest.mark.parametrize("missing", (("_cuda_getCurrentRawStream",), ("_cuda_getDevice",), ("_cuda_getCurrentRawStream", "_cuda_getDevice")))
def test_public_call_where_the_private_ones_are_missing(monkeypatch, missing):
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.setattr(torch._C, name, lambda *a: pytest.fail("half of the private calls is of no use"), raising=False)
    for name in missing:
        monkeypatch.delattr(torch._C, name)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream(0x1234))
    assert B._stream_ptr(None) == 0x1234


def test_private_calls(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x5000 + device, raising=False)
    assert B._stream_ptr(None) == 0x5003
    assert B._stream_ptr(Stream(0x77)) == 0x77
