"""Argument marshalling of the binding (csrc/marshal.cpp): what is taken, what is refused and with which error, and the stream
that a call without a stream argument goes to."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2010_00704_amd import binding as B

FAKE = 64                                    # an address that no refused call touches


class Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("call,want", [
    (lambda d: B.bcnn_conv2d_binary(d, FAKE, FAKE, 2 * FAKE, 0), B.BCNN_ERR_UNSUPPORTED),
    (lambda d: B.bcnn_conv2d_binary((1, 64, 5, 5, 64, 5, 5, 1, 1), FAKE, FAKE, y=2 * FAKE, stream=0), B.BCNN_ERR_UNSUPPORTED),
    (lambda d: B.bcnn_conv2d_binary_variant(d, FAKE, FAKE, None, 2 * FAKE, np.int64(0), 0), B.BCNN_ERR_UNSUPPORTED),
    (lambda d: B.bcnn_pack(None, 0, 1, 1, 1, FAKE, 0), B.BCNN_ERR_INVALID_ARG),
    (lambda d: B.bcnn_pack(FAKE, np.int64(0), 1, True, 0, 2 * FAKE, 0), B.BCNN_ERR_INVALID_ARG),
    (lambda d: B.bcnn_pack(FAKE, 0, 2 ** 70, 1, 1, 2 * FAKE, 0), B.BCNN_ERR_INVALID_ARG),       # cut to 64 bits: no images
    (lambda d: B.bcnn_pack(torch.zeros(4).as_subclass(Sub), 0, 1, 0, 1, FAKE, 0), B.BCNN_ERR_INVALID_ARG),
    (lambda d: B.bcnn_pack(torch.nn.Parameter(torch.zeros(4)), 0, 1, 0, 1, FAKE, 0), B.BCNN_ERR_INVALID_ARG),
    (lambda d: B.bcnn_conv2d_binary_module(d, FAKE, FAKE, FAKE, FAKE, None, None, None, 0, FAKE, None, stream=0), B.BCNN_ERR_UNSUPPORTED),
    (lambda d: B.bcnn_pack(torch.zeros(4, 4).t(), 0, 1, 1, 1, FAKE, 0), ValueError),
    (lambda d: B.bcnn_pack(torch.zeros(4, 4).as_subclass(Sub).t(), 0, 1, 1, 1, FAKE, 0), ValueError),
    (lambda d: B.bcnn_pack("x", 0, 1, 1, 1, FAKE, 0), AttributeError),
    (lambda d: B.bcnn_pack(FAKE, 0, 1, 0, 1, 2 * FAKE, "s"), AttributeError),
    (lambda d: B.bcnn_pack(FAKE, 0, 1.5, 1, 1, 2 * FAKE, 0), ctypes.ArgumentError),
    (lambda d: B.bcnn_conv2d_binary(None, FAKE, FAKE, 2 * FAKE, 0), TypeError),
    (lambda d: B.bcnn_conv2d_binary_variant(d, FAKE, FAKE, None, 2 * FAKE, "a", 0), ValueError),
])
def test_taken_and_refused(call, want):
    desc = B.conv_desc(1, 64, 5, 5, 64, 5, 1, 1)     # a filter size that no kernel takes: nothing is launched
    if isinstance(want, int):
        assert call(desc) == want
    else:
        with pytest.raises(want):
            call(desc)


@pytest.mark.gpu
def test_calls_without_a_stream_follow_torch():
    """Captured on a side stream, called without a stream argument: the graph holds the call, and replays it on new inputs."""
    assert torch.cuda.is_available()
    x = torch.randn((3, 40, 9, 7), device="cuda")
    out, want = (torch.empty((3 * 63, 2), dtype=torch.int32, device="cuda") for _ in range(2))
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        B.check(B.bcnn_pack(x, B.BCNN_F32, 3, 40, 63, out))
    for _ in range(3):
        x.copy_(torch.randn_like(x))
        out.fill_(77)
        graph.replay()
        B.check(B.bcnn_pack(x, B.BCNN_F32, 3, 40, 63, want, stream=torch.cuda.current_stream()))
        torch.cuda.synchronize()
        assert torch.equal(out, want)
