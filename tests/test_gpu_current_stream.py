"""Calls without a stream go to torch's current stream of the current device."""
import pytest
import torch

from paper_2406_02542_amd import api

pytestmark = pytest.mark.gpu


def test_current_stream():
    torch.zeros(1, device="cuda")
    assert api._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert api._stream_ptr(None) == side.cuda_stream
        assert api._stream_ptr(other) == other.cuda_stream
        graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert api._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
        torch.zeros(1, device="cuda")
    assert api._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
