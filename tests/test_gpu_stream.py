"""Calls without a stream argument go to torch's current stream: of the thread, inside stream contexts, and in graph
capture (where a launch on any other stream would fail the capture)."""
import threading

import pytest
import torch

from paper_2010_00704_amd import binding as B
from gpu_helpers import gpu_device

pytestmark = pytest.mark.gpu


def test_default_stream_is_the_current_one():
    dev = gpu_device()
    same = lambda: B._stream(None) == torch.cuda.current_stream().cuda_stream  # noqa: E731
    assert same()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert same() and B._stream(None) == side.cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append(same()))     # another thread has its own current stream
        t.start()
        t.join()
        assert seen == [True]
    assert same()
    src = torch.arange(256, dtype=torch.int32, device=dev)
    dst = torch.zeros_like(src)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        B.check(B.bcnn_diag_copy_u32(src, dst, 256), "copy")
    for k in range(3):
        src.add_(k)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(src, dst)
