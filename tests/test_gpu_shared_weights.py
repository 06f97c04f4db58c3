"""The direct kernel's form whose workgroups share expanded weights: every tile and width of its loads, for each kind of
output, against the vector-ALU kernels (which the other tests hold against the oracle).  Pixels, channels and words are
ragged; operands lie a word past an allocation's start, so that the staged kernel covers none of these calls.  Which tile and
width a call takes is checked on the host, from the same list, by test_host_shared_plan.py."""
import pytest
import torch

from paper_2010_00704_amd import binding as B
from gpu_helpers import gpu_device
from test_gpu_direct_tiles import Draw, both

pytestmark = pytest.mark.gpu

S_1X1, S_2X1, S_2X2 = 1, 2, 3                          # tiles: csrc/shared_plan.h
BITS, SUMS, HALF, FLOAT = 0, 1, 2, 3

CONVS = [
    # kind, tile, words per load, (n, c_in, h, w, c_out, filter, stride)
    (BITS, S_1X1, 1, (13, 20, 27, 26, 33, 1, 1)),
    (BITS, S_1X1, 2, (7, 75, 27, 26, 200, 1, 1)),
    (BITS, S_1X1, 3, (101, 330, 27, 27, 33, 1, 2)),
    (BITS, S_1X1, 4, (101, 200, 27, 27, 70, 3, 2)),
    (BITS, S_1X1, 5, (101, 260, 27, 27, 33, 1, 2)),
    (BITS, S_2X1, 1, (101, 20, 27, 27, 33, 1, 2)),
    (BITS, S_2X1, 2, (101, 75, 27, 27, 33, 1, 2)),
    (BITS, S_2X1, 3, (61, 330, 27, 26, 100, 1, 2)),
    (BITS, S_2X1, 4, (61, 200, 27, 26, 33, 1, 1)),
    (BITS, S_2X1, 5, (29, 260, 27, 27, 33, 1, 1)),
    (BITS, S_2X2, 1, (101, 20, 27, 27, 70, 1, 1)),
    (BITS, S_2X2, 2, (101, 75, 27, 27, 70, 1, 1)),
    (BITS, S_2X2, 3, (101, 140, 27, 27, 70, 1, 1)),
    (BITS, S_2X2, 4, (101, 200, 27, 27, 70, 1, 1)),
    (BITS, S_2X2, 5, (101, 260, 27, 27, 70, 1, 1)),
    (SUMS, S_1X1, 3, (101, 140, 27, 27, 70, 3, 2)),
    (SUMS, S_1X1, 4, (61, 420, 27, 26, 70, 3, 1)),
    (SUMS, S_1X1, 5, (61, 260, 27, 26, 200, 3, 2)),
    (SUMS, S_2X1, 1, (101, 50, 27, 27, 100, 3, 1)),
    (SUMS, S_2X1, 2, (29, 110, 27, 27, 300, 3, 1)),
    (SUMS, S_2X1, 3, (101, 140, 27, 27, 33, 3, 1)),
    (SUMS, S_2X1, 4, (61, 200, 27, 26, 100, 3, 1)),
    (SUMS, S_2X1, 5, (101, 260, 27, 27, 33, 3, 1)),
    (SUMS, S_2X2, 1, (101, 50, 27, 27, 300, 3, 1)),
    (SUMS, S_2X2, 2, (101, 110, 27, 27, 130, 3, 1)),
    (SUMS, S_2X2, 3, (61, 140, 27, 26, 200, 3, 1)),
    (SUMS, S_2X2, 4, (101, 200, 27, 27, 100, 3, 1)),
    (SUMS, S_2X2, 5, (61, 260, 27, 26, 130, 3, 1)),
    (HALF, S_1X1, 2, (101, 110, 27, 27, 70, 3, 2)),
    (HALF, S_1X1, 3, (101, 140, 27, 27, 70, 3, 2)),
    (HALF, S_1X1, 4, (61, 200, 27, 26, 33, 3, 1)),
    (HALF, S_1X1, 5, (101, 260, 27, 27, 70, 3, 2)),
    (HALF, S_2X1, 1, (101, 50, 27, 27, 100, 3, 1)),
    (HALF, S_2X1, 2, (61, 110, 27, 26, 100, 3, 1)),
    (HALF, S_2X1, 3, (101, 140, 27, 27, 33, 3, 1)),
    (HALF, S_2X1, 4, (101, 200, 27, 27, 33, 3, 1)),
    (HALF, S_2X1, 5, (101, 260, 27, 27, 33, 3, 1)),
    (FLOAT, S_1X1, 3, (61, 140, 27, 26, 33, 3, 1)),
    (FLOAT, S_1X1, 4, (61, 200, 27, 26, 33, 3, 1)),
    (FLOAT, S_1X1, 5, (61, 260, 27, 26, 200, 3, 2)),
    (FLOAT, S_2X1, 3, (101, 140, 27, 27, 300, 3, 2)),
    (FLOAT, S_2X1, 4, (101, 420, 27, 27, 100, 3, 1)),
    (FLOAT, S_2X1, 5, (101, 260, 27, 27, 300, 3, 2)),
]


def module_parts(form):
    return "id" in form, "r" in form, "x" in form


@pytest.mark.parametrize("kind,tile,wide,shape", CONVS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_tile(kind, tile, wide, shape):
    gpu_device()
    n, c, h, w, o, k, stride = shape
    d = Draw(83000 + 17 * c + o + kind)
    (x, _, keep_x), (wt, _, keep_w) = d.packed(n, c, h, w), d.packed(o, c, k, k)
    desc = B.conv_desc(n, c, h, w, o, k, stride, k // 2)
    ho, wo = B.out_shape(desc)
    m, words, total = n * ho * wo, (o + 31) // 32, c * k * k
    if kind == BITS:
        thr = d.real((o,), total ** 0.5).to(torch.int32)
        ends = torch.tensor([-2 ** 31, 2 ** 31 - 1, -total, total, total + 1], dtype=torch.int32, device="cuda")
        thr[:5] = ends                                  # thresholds that every sum, and none, reaches
        both(lambda out, v: B.bcnn_conv2d_binary_variant(desc, x, wt, thr, out[0], v), [((m, words), torch.int32)])
    elif kind == SUMS:
        both(lambda out, v: B.bcnn_conv2d_binary_variant(desc, x, wt, None, out[0], v), [((m, o), torch.int32)])
    else:
        g, b, slope, nxt = d.real((o,), 4 / total ** 0.5), d.real((o,), 3.0), d.real((o,), 1.0), d.real((o,), 5.0)
        types = [(torch.float32, B.BCNN_F32)] if kind == FLOAT else [(torch.float16, B.BCNN_F16), (torch.bfloat16, B.BCNN_BF16)]
        for dtype, code in types:
            ident = d.real((m, o), 30.0).to(dtype)
            for has_id, has_r, has_x in ((1, 1, 1), (0, 1, 1), (1, 0, 1), (1, 1, 0)):
                both(lambda out, v: B.bcnn_conv2d_binary_module(desc, x, wt, g, b, ident if has_id else None, slope, nxt, code,
                                                                out[0] if has_r else None, out[1] if has_x else None, v),
                     [((m, o), dtype), ((m, words), torch.int32)])
    del keep_x, keep_w
