"""Calls without a stream argument go to torch's current stream of the calling thread."""
import threading

import pytest
import torch

from paper_2605_06676_amd import lkv

pytestmark = pytest.mark.gpu


def handle(stream=None):
    return lkv._stream_ptr(stream).value or 0


def test_the_current_stream_of_the_thread():
    default, side = torch.cuda.current_stream().cuda_stream, torch.cuda.Stream()
    assert handle() == default and handle(side) == side.cuda_stream
    with torch.cuda.stream(side):
        assert handle() == side.cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append(handle()))   # the other thread's current stream is the default one
        t.start()
        t.join()
        assert seen == [default]
    assert handle() == default
    with torch.cuda.graph(torch.cuda.CUDAGraph()):
        assert handle() == torch.cuda.current_stream().cuda_stream != default
        torch.zeros(1, device="cuda")


def test_without_the_short_way(monkeypatch):
    monkeypatch.setattr(lkv, "_current_stream", None)
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert handle() == side.cuda_stream
