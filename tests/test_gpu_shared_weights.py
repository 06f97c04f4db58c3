"""The direct kernel's form whose workgroups share expanded weights: every tile and width of its loads, for each kind of
output, and in branch mode also the forms whose waves take whole taps or their own operands, against the vector-ALU kernels (which the other tests hold against the oracle).  Pixels, channels and words are
ragged; operands lie a word past an allocation's start, so that the staged kernel covers none of these calls (but ALIGNED).  Which tile and
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
    (HALF, S_1X1, 3, (101, 140, 27, 27, 70, 3, 2)),
    (HALF, S_1X1, 4, (61, 200, 27, 26, 33, 3, 1)),
    (HALF, S_1X1, 5, (101, 260, 27, 27, 70, 3, 2)),
    (HALF, S_2X1, 1, (101, 50, 27, 27, 100, 3, 1)),
    (HALF, S_2X1, 2, (61, 75, 27, 26, 339, 3, 1)),
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

# modules of whole 128-channel tiles and 16-byte aligned operands, which the staged kernel covers as well
ALIGNED = [
    (HALF, S_1X1, 2, (39, 128, 14, 14, 640, 3, 1)),
    (FLOAT, S_1X1, 2, (46, 128, 14, 14, 640, 3, 1)),
]

OWN, APART, SHARED = 0, 1, 2                           # branch forms; tile 1 of APART: four waves a block
T_2X1, T_1X1, T_2X2 = 3, 4, 5                          # tiles of OWN: csrc/direct_plan.h
OUTS = ["bits", "f32", "module_f32", "module_f16"]
BRANCHES = [
    # form, tile, words per load, output, (n, c_in, h, w, c_out, branches): nine taps of a 3x3 filter, or parallel ones
    (APART, 1, 1, "bits", (1, 20, 9, 7, 33, 9)),
    (APART, 1, 2, "f32", (1, 75, 9, 7, 33, 9)),
    (APART, 1, 3, "module_f16", (2, 140, 13, 11, 70, 9)),
    (APART, 1, 4, "module_f32", (1, 200, 9, 7, 33, 9)),
    (APART, 1, 4, "bits", (1, 420, 9, 7, 33, 9)),
    (APART, 1, 5, "f32", (1, 260, 9, 7, 33, 3)),
    (APART, 1, 1, "module_f16", (1, 50, 9, 7, 36, 3)),
    (OWN, T_2X1, 1, "module_f32", (209, 50, 27, 27, 100, 3)),
    (OWN, T_2X1, 2, "module_f32", (209, 75, 27, 27, 100, 1)),
    (OWN, T_2X1, 1, "module_f16", (19, 20, 27, 27, 1000, 1)),
    (OWN, T_2X2, 1, "bits", (209, 20, 27, 27, 33, 8)),
    (OWN, T_2X2, 1, "f32", (209, 20, 27, 27, 36, 8)),
    (OWN, T_2X2, 1, "module_f16", (209, 50, 27, 27, 100, 3)),
    (OWN, T_2X2, 2, "module_f16", (209, 110, 27, 27, 100, 1)),
    (SHARED, S_1X1, 1, "bits", (1, 20, 9, 7, 33, 16)),
    (SHARED, S_1X1, 2, "f32", (1, 75, 9, 7, 33, 16)),
    (SHARED, S_1X1, 3, "module_f16", (1, 140, 9, 7, 33, 16)),
    (SHARED, S_1X1, 4, "module_f32", (1, 200, 9, 7, 33, 16)),
    (SHARED, S_1X1, 5, "bits", (1, 260, 9, 7, 33, 16)),
    (SHARED, S_2X1, 2, "f32", (61, 75, 27, 26, 100, 3)),
    (SHARED, S_2X1, 3, "bits", (61, 140, 27, 26, 100, 3)),
    (SHARED, S_2X1, 4, "f32", (61, 200, 27, 26, 100, 3)),
    (SHARED, S_2X1, 5, "bits", (61, 260, 27, 26, 100, 3)),
    (SHARED, S_2X1, 3, "module_f32", (133, 140, 27, 26, 100, 9)),
    (SHARED, S_2X1, 4, "module_f32", (133, 200, 27, 26, 100, 9)),
    (SHARED, S_2X1, 5, "module_f32", (101, 260, 27, 26, 100, 9)),
]
BRANCHES += [(OWN, T_1X1, wide, out, (19, c, 27, 27, 33, taps)) for wide, c, taps in ((1, 20, 3), (1, 50, 2), (2, 75, 1), (2, 110, 1)) for out in OUTS]
BRANCHES += [(SHARED, S_1X1, wide, out, (13, c, 27, 26, 70, 9)) for wide, c in ((1, 20), (2, 75), (3, 140), (4, 200), (5, 260)) for out in OUTS]
BRANCHES += [(SHARED, S_2X1, wide, out, (61, c, 27, 26, 100, 9)) for wide, c in ((1, 50), (2, 110), (3, 170), (4, 230), (5, 290))
             for out in ("bits", "f32", "module_f16")]


@pytest.mark.parametrize("kind,tile,wide,shape", CONVS + ALIGNED, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_tile(kind, tile, wide, shape):
    gpu_device()
    n, c, h, w, o, k, stride = shape
    d = Draw(83000 + 17 * c + o + kind)
    (x, _, keep_x), (wt, _, keep_w) = d.packed(n, c, h, w), d.packed(o, c, k, k)
    if (kind, tile, wide, shape) in ALIGNED:
        keep_x, keep_w = keep_x[1:].clone(), keep_w[1:].clone()
        x, wt = keep_x.data_ptr(), keep_w.data_ptr()
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


@pytest.mark.parametrize("pad_mode", ["minus", "words", "zero"])
@pytest.mark.parametrize("form,tile,wide,out,shape", BRANCHES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_branch_form(form, tile, wide, out, shape, pad_mode):
    gpu_device()
    n, c, h, w, o, taps = shape
    k = 3 if taps == 9 else 1
    d = Draw(84000 + 17 * c + n)
    own = taps in (1, 3)                                # parallel branches of their own tensors, or of one
    (x, _, keep_x), (wt, _, keep_w), (pad, _, keep_p) = d.packed(n * (taps if own else 1), c, h, w), d.packed(o, c, taps), d.packed(taps, c, 1)
    desc = B.conv_desc(n, c, h, w, o, k, 1, k // 2)
    m, words = n * h * w, (o + 31) // 32
    scale, bias = d.real((taps, o), 4 / (taps * c) ** 0.5), d.real((o,), 3.0)
    scale[:, 0], bias[1] = float("inf"), float("nan")   # sums of infinities and no numbers: their sign bits too
    args = (desc, taps, x, m * ((c + 31) // 32) if own else 0, wt, pad if pad_mode == "words" else None,
            B.BCNN_PAD_ZERO if pad_mode == "zero" else B.BCNN_PAD_WORDS, scale, bias if out != "f32" else None)
    if out == "bits":
        both(lambda z, v: B.bcnn_conv2d_binary_branches_sign_pack(*args, z[0], v), [((m, words), torch.int32)])
    elif out == "f32":
        scale[:, 0] = 0.25
        both(lambda z, v: B.bcnn_conv2d_binary_branches(*args, z[0], v), [((m, o), torch.float32)])
    else:
        scale[:, 0], bias[1] = 0.25, 0.5
        dtype, code = (torch.float16, B.BCNN_F16) if out == "module_f16" else (torch.float32, B.BCNN_F32)
        ident, slope, nxt = d.real((m, o), 30.0).to(dtype), d.real((o,), 1.0), d.real((o,), 5.0)
        both(lambda z, v: B.bcnn_conv2d_binary_branches_module(*args, ident, slope, nxt, code, z[0], z[1], v),
             [((m, o), dtype), ((m, words), torch.int32)])
    del keep_x, keep_w, keep_p
