"""The binding runs on torch's current stream, inside and outside a stream
context and under graph capture, as on a stream that is passed."""

import pytest

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    import torch
    from paper_2412_02962_amd import pcpp
    torch.cuda.init()
    handle = lambda: torch.cuda.current_stream().cuda_stream
    assert pcpp._stream(None) == handle()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert pcpp._stream(None) == handle() == side.cuda_stream
    assert pcpp._stream(None) == handle()
    assert pcpp._stream(side) == side.cuda_stream
    graph = torch.cuda.CUDAGraph()
    x = torch.zeros(4, device="cuda:0")
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        captured = (pcpp._stream(None), handle())
        x.add_(1)
    assert captured[0] == captured[1] != handle()
