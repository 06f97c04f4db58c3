"""Every tile of the direct matrix-core kernel with every walk of K that AUTO reaches, for each kind of output, and padded branch
calls of every output, against the vector-ALU kernels (which the other tests hold against the oracle).  Operands lie a word past
an allocation's start, so that the staged kernel covers none of these calls; pixels and channels are ragged.  Which tile a plain
call takes is checked on the host, from the same list, by test_host_direct_plan.py; the forms of branch calls and their
tiles are test_gpu_shared_weights.py's."""
import pytest
import torch

from paper_2010_00704_amd import binding as B
from gpu_helpers import gpu_device

pytestmark = pytest.mark.gpu

K4_1X1, K4_2X2, T_2X1, T_1X1 = 1, 2, 3, 4               # tiles: csrc/direct_plan.h
UNITS, TAIL, WORDS = 0, 1, 2                            # walks of K
BITS, SUMS, HALF, FLOAT = 0, 1, 2, 3

CONVS = [
    # kind, tile, walk, (n, c_in, h, w, c_out, filter)
    (BITS, K4_1X1, UNITS, (1, 120, 5, 7, 33, 1)),
    (BITS, K4_1X1, TAIL, (1, 150, 5, 7, 33, 1)),
    (BITS, K4_1X1, WORDS, (1, 20, 5, 7, 33, 3)),
    (BITS, K4_2X2, UNITS, (33, 380, 28, 28, 33, 3)),
    (BITS, K4_2X2, TAIL, (33, 410, 28, 28, 33, 3)),
    (BITS, T_1X1, UNITS, (9, 125, 27, 27, 33, 1)),
    (BITS, T_1X1, TAIL, (9, 150, 27, 27, 33, 1)),
    (BITS, T_1X1, WORDS, (9, 90, 27, 27, 33, 1)),
    (SUMS, K4_1X1, UNITS, (1, 120, 5, 7, 33, 1)),
    (SUMS, K4_1X1, TAIL, (1, 150, 5, 7, 34, 1)),
    (SUMS, K4_1X1, WORDS, (1, 20, 5, 7, 35, 3)),
    (SUMS, K4_2X2, UNITS, (49, 380, 28, 28, 33, 3)),
    (SUMS, K4_2X2, TAIL, (49, 270, 28, 28, 36, 3)),
    (SUMS, T_2X1, UNITS, (97, 630, 28, 28, 33, 1)),
    (SUMS, T_2X1, TAIL, (129, 270, 28, 28, 34, 1)),
    (SUMS, T_2X1, WORDS, (97, 50, 28, 28, 33, 3)),
    (SUMS, T_1X1, UNITS, (5, 125, 26, 27, 130, 1)),
    (SUMS, T_1X1, TAIL, (5, 150, 26, 27, 131, 1)),
    (SUMS, T_1X1, WORDS, (5, 30, 26, 27, 130, 1)),
    (HALF, K4_1X1, UNITS, (1, 380, 5, 7, 36, 1)),
    (HALF, K4_1X1, TAIL, (1, 270, 5, 7, 33, 1)),
    (HALF, K4_1X1, WORDS, (1, 20, 5, 7, 36, 3)),
    (HALF, K4_2X2, UNITS, (33, 500, 28, 28, 36, 3)),
    (HALF, K4_2X2, TAIL, (33, 410, 28, 28, 33, 3)),
    (HALF, T_2X1, UNITS, (129, 125, 28, 28, 36, 3)),
    (HALF, T_2X1, TAIL, (275, 270, 28, 28, 33, 1)),
    (HALF, T_2X1, WORDS, (275, 20, 28, 28, 33, 3)),
    (HALF, T_1X1, UNITS, (49, 380, 28, 28, 36, 1)),
    (HALF, T_1X1, TAIL, (49, 270, 28, 28, 33, 1)),
    (HALF, T_1X1, WORDS, (49, 20, 28, 28, 36, 3)),
    (FLOAT, K4_1X1, UNITS, (1, 380, 5, 7, 36, 1)),
    (FLOAT, K4_1X1, TAIL, (1, 270, 5, 7, 33, 1)),
    (FLOAT, K4_1X1, WORDS, (1, 20, 5, 7, 36, 3)),
    (FLOAT, K4_2X2, UNITS, (33, 500, 28, 28, 36, 3)),
    (FLOAT, K4_2X2, TAIL, (33, 410, 28, 28, 33, 3)),
    (FLOAT, T_2X1, UNITS, (129, 125, 28, 28, 36, 3)),
    (FLOAT, T_2X1, TAIL, (275, 270, 28, 28, 33, 1)),
    (FLOAT, T_2X1, WORDS, (97, 50, 28, 28, 100, 3)),
    (FLOAT, T_1X1, UNITS, (49, 380, 28, 28, 36, 1)),
    (FLOAT, T_1X1, TAIL, (49, 270, 28, 28, 33, 1)),
    (FLOAT, T_1X1, WORDS, (49, 20, 28, 28, 36, 3)),
]
BRANCHES = [
    # output, (n, c_in, h, w, c_out, branches): nine taps of a 3x3 filter, or parallel ones
    (out, (n, c, 28, 28, 100 if n > 9 else 36, 9))
    for c in (30, 220, 288)             # one word, seven (single words only), nine (a group and a single word)
    for n in (9, 97) for out in ("bits", "f32", "module_f32", "module_f16")
] + [("module_f16", (64, 1010, 28, 28, 100, 16))]


class Draw:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def real(self, shape, bound):
        return (torch.rand(shape, generator=self.gen, device="cuda") * 2 - 1) * bound

    def packed(self, *shape):
        """+-1 in [outer, channels, spatial], packed, a word past an allocation's start: (address, words, owner)."""
        x = torch.where(torch.rand(shape, generator=self.gen, device="cuda") < 0.5, 1, -1).to(torch.int8)
        words = B.pack_nchw(x).reshape(-1)
        owner = torch.zeros(words.numel() + 8, dtype=torch.int32, device="cuda")
        owner[1:1 + words.numel()] = words
        return owner.data_ptr() + 4, words.numel(), owner


def same(a, b):
    return torch.equal(a.reshape(-1).view(torch.uint8), b.reshape(-1).view(torch.uint8))


def banded(shape, dtype):
    """An output of rows between bands of 32 rows and more: (the whole buffer, the output in it, at an allocation's alignment)."""
    rows, row = shape
    band = (32 * row + 255) // 256 * 256
    whole = torch.full((2 * band + rows * row,), 77, dtype=dtype, device="cuda")
    return whole, whole[band:band + rows * row].view(shape)


def both(call, outputs):
    """The call under AUTO and on the vector ALUs: every output the same, to the bit, and neither writes around it."""
    got = []
    for variant in (B.BCNN_VARIANT_AUTO, B.BCNN_VARIANT_VALU):
        out = [banded(shape, dtype) for shape, dtype in outputs]
        B.check(call([part for _, part in out], variant))
        got.append(out)
    torch.cuda.synchronize()
    for (a, inside_a), (b, inside_b) in zip(*got):
        assert same(inside_a, inside_b)
        for whole, inside in ((a, inside_a), (b, inside_b)):
            band = (whole.numel() - inside.numel()) // 2
            assert (whole[:band] == 77).all() and (whole[-band:] == 77).all(), "write around the output"


@pytest.mark.parametrize("kind,tile,walk,shape", CONVS, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_tile(kind, tile, walk, shape):
    gpu_device()
    n, c, h, w, o, k = shape
    d = Draw(81000 + 17 * c + o + kind)
    (x, _, keep_x), (wt, _, keep_w) = d.packed(n, c, h, w), d.packed(o, c, k, k)
    desc = B.conv_desc(n, c, h, w, o, k, 1, k // 2)
    m, words, total = n * h * w, (o + 31) // 32, c * k * k
    if kind == BITS:
        thr = (d.real((o,), total ** 0.5)).to(torch.int32)
        both(lambda out, v: B.bcnn_conv2d_binary_variant(desc, x, wt, thr, out[0], v), [((m, words), torch.int32)])
    elif kind == SUMS:
        both(lambda out, v: B.bcnn_conv2d_binary_variant(desc, x, wt, None, out[0], v), [((m, o), torch.int32)])
    else:
        g, b, slope, nxt = d.real((o,), 4 / total ** 0.5), d.real((o,), 3.0), d.real((o,), 1.0), d.real((o,), 5.0)
        for dtype, code in [(torch.float32, B.BCNN_F32)] if kind == FLOAT else [(torch.float16, B.BCNN_F16), (torch.bfloat16, B.BCNN_BF16)]:
            ident = d.real((m, o), 30.0).to(dtype)
            both(lambda out, v: B.bcnn_conv2d_binary_module(desc, x, wt, g, b, ident, slope, nxt, code, out[0], out[1], v),
                 [((m, o), dtype), ((m, words), torch.int32)])
    del keep_x, keep_w


@pytest.mark.parametrize("pad_mode", ["minus", "words", "zero"])
@pytest.mark.parametrize("out,shape", BRANCHES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_padded_branches(out, shape, pad_mode):
    gpu_device()
    n, c, h, w, o, taps = shape
    k = 3 if taps == 9 else 1
    d = Draw(82000 + 17 * c + n)
    (x, _, keep_x), (wt, _, keep_w), (pad, _, keep_p) = d.packed(n, c, h, w), d.packed(o, c, taps), d.packed(taps, c, 1)
    desc = B.conv_desc(n, c, h, w, o, k, 1, k // 2)
    m, words = n * h * w, (o + 31) // 32
    scale, bias = d.real((taps, o), 4 / (taps * c) ** 0.5), d.real((o,), 3.0)
    args = (desc, taps, x, 0, wt, pad if pad_mode == "words" else None,
            B.BCNN_PAD_ZERO if pad_mode == "zero" else B.BCNN_PAD_WORDS, scale, bias)
    if out == "bits":
        both(lambda z, v: B.bcnn_conv2d_binary_branches_sign_pack(*args, z[0], v), [((m, words), torch.int32)])
    elif out == "f32":
        both(lambda z, v: B.bcnn_conv2d_binary_branches(*args, z[0], v), [((m, o), torch.float32)])
    else:
        dtype, code = (torch.float16, B.BCNN_F16) if out == "module_f16" else (torch.float32, B.BCNN_F32)
        ident, slope, nxt = d.real((m, o), 30.0).to(dtype), d.real((o,), 1.0), d.real((o,), 5.0)
        both(lambda z, v: B.bcnn_conv2d_binary_branches_module(*args, ident, slope, nxt, code, z[0], z[1], v),
             [((m, o), dtype), ((m, words), torch.int32)])
    del keep_x, keep_w, keep_p
