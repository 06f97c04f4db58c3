"""The matrix-core kernels whose weights stay in LDS, against the vector-ALU kernels (which the other tests hold against the oracle):
every width of its loads, odd and even numbers of groups, taps whose words do not fill their groups, channels that do not fill
a word, a channel tile or a block, ragged last columns, passes of one to four columns, several tables of places, both strides, no padding;
in branch mode odd and even numbers of taps, pad words, tensors of their own, no bias, infinities and NaN.
That these calls take the kernels is checked on the host, from the same list, by test_host_resident_plan.py."""
import pytest
import torch

from paper_2010_00704_amd import binding as B
from gpu_helpers import gpu_device
from test_gpu_direct_tiles import Draw, both

pytestmark = pytest.mark.gpu

CALLS = [
    # words per load, (n, c_in, h, w, c_out, stride, pad)
    (3, (34, 140, 27, 26, 190, 1, 1)),          # 5 words: halves of 3 and 2
    (3, (95, 192, 27, 26, 64, 1, 1)),           # 6 words, all whole
    (4, (34, 200, 29, 28, 161, 1, 0)),          # 7 words, part of the last
    (4, (70, 256, 14, 14, 320, 1, 1)),          # 8 words, all whole
    (5, (30, 320, 27, 27, 200, 1, 1)),          # 10 words, all whole
    (5, (160, 290, 29, 27, 100, 2, 1)),          # the same, part of the last
    (3, (48, 380, 27, 26, 128, 1, 1)),          # 12 words in two groups a tap
    (4, (107, 500, 27, 26, 250, 2, 0)),          # 16 words in two groups, part of the last
    (4, (64, 512, 14, 14, 512, 1, 1)),          # as many K-steps as LDS holds
    (4, (5, 224, 11, 13, 7000, 1, 1)),          # few columns, many channel tiles: passes of one or two
    (3, (600, 129, 27, 28, 60, 1, 1)),          # 55 columns and more a workgroup: two tables of places
]

OUTS = ("bits", "f32")
BRANCHES = [
    # words per load, (n, c_in, h, w, c_out, taps, stride)
    (3, (13, 140, 27, 26, 190, 9, 1)),
    (4, (30, 200, 27, 26, 161, 9, 1)),
    (4, (70, 256, 28, 28, 64, 9, 2)),
    (5, (13, 320, 27, 27, 200, 9, 1)),
    (5, (61, 290, 27, 26, 33, 9, 1)),
    (4, (300, 224, 28, 27, 50, 9, 1)),          # more columns a workgroup than its table of places holds
    (3, (61, 192, 27, 26, 100, 4, 1)),
    (4, (61, 256, 27, 26, 100, 16, 1)),
    (5, (40, 300, 27, 26, 100, 7, 2)),
    (3, (30, 130, 27, 26, 170, 5, 1)),          # (up to five taps and tensors of their own: bits only)
    (3, (61, 192, 27, 26, 100, 6, 1)),
] + [(wide, (61, c, 27, 26, 100, taps, 1)) for wide, c, taps in ((4, 250, 1), (3, 180, 2), (5, 260, 3))]
# what these kernels leave to the form with shared weights: taps of two loads
BRANCHES_OF_TWO_LOADS = [(3, (61, 380, 27, 26, 100, 9, 1)), (4, (61, 500, 27, 26, 100, 9, 1)), (5, (61, 630, 27, 26, 100, 9, 1)), (5, (61, 260, 27, 26, 100, 2, 1))]


def own_tensors(taps):
    """Whether a call of the list gives each of its branches a tensor of its own."""
    return taps in (3, 4, 7)


@pytest.mark.parametrize("wide,shape", CALLS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_bits(wide, shape):
    gpu_device()
    n, c, h, w, o, stride, pad = shape
    d = Draw(91000 + 17 * c + o)
    (x, _, keep_x), (wt, _, keep_w) = d.packed(n, c, h, w), d.packed(o, c, 3, 3)
    desc = B.conv_desc(n, c, h, w, o, 3, stride, pad)
    m = n * ((h + 2 * pad - 3) // stride + 1) * ((w + 2 * pad - 3) // stride + 1)
    thr = d.real((o,), (9 * c) ** 0.5).to(torch.int32)
    thr[0], thr[-1] = -2 ** 31, 2 ** 31 - 1                # out of reach: bits of one kind
    both(lambda out, v: B.bcnn_conv2d_binary_variant(desc, x, wt, thr, out[0], v), [((m, (o + 31) // 32), torch.int32)])
    del keep_x, keep_w


@pytest.mark.parametrize("pad_mode", ["words", "minus"])
@pytest.mark.parametrize("out", OUTS)
@pytest.mark.parametrize("wide,shape", BRANCHES + BRANCHES_OF_TWO_LOADS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_branches(wide, shape, out, pad_mode):
    gpu_device()
    n, c, h, w, o, taps, stride = shape
    k = 3 if taps == 9 else 1
    d = Draw(92000 + 17 * c + o + taps)
    own = own_tensors(taps)
    (x, _, keep_x), (wt, _, keep_w), (pad, _, keep_p) = d.packed(n * (taps if own else 1), c, h, w), d.packed(o, c, taps), d.packed(taps, c, 1)
    desc = B.conv_desc(n, c, h, w, o, k, stride, k // 2)
    ho, wo = B.out_shape(desc)
    m, words = n * ho * wo, (o + 31) // 32
    scale, bias = d.real((taps, o), 4 / (taps * c) ** 0.5), d.real((o,), 3.0)
    bias[2] = -0.0
    scale[:, 2] = 0.0                                   # a sum of zeros: which one decides the float, not the bit
    if out == "bits":
        scale[:, 0], bias[1] = float("inf"), float("nan")
    args = (desc, taps, x, n * h * w * ((c + 31) // 32) if own else 0, wt, pad if pad_mode == "words" else None, B.BCNN_PAD_WORDS, scale,
            bias if taps % 4 else None)
    if out == "bits":
        both(lambda z, v: B.bcnn_conv2d_binary_branches_sign_pack(*args, z[0], v), [((m, words), torch.int32)])
    else:
        both(lambda z, v: B.bcnn_conv2d_binary_branches(*args, z[0], v), [((m, o), torch.float32)])
    del keep_x, keep_w, keep_p
