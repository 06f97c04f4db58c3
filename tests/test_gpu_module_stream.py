"""1x1 modules of up to 256 input channels with every part present (the streaming kernel), against the oracle: words per
pixel 1 to 8 (odd ones too), channel counts around 32, 64 and 128 with partial words, pixels around a block of 32,
stride 2, a replicated identity, in place, all three stream types."""
import numpy as np
import pytest
import torch

import oracle
from paper_2010_00704_amd import binding as B
from paper_2010_00704_amd import workloads as W
from gpu_helpers import Guarded, REAL_IDS, REAL_PARAMS, gpu_device, i32, real_code, real_np_dtype, real_store, real_values, up

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, c_in, h, w, c_out, stride, identity channels
    (1, 8, 1, 1, 8, 1, 8),
    (1, 32, 5, 7, 32, 1, 32),
    (3, 64, 31, 1, 64, 1, 64),
    (1, 96, 9, 7, 104, 1, 104),          # three words: one K-step more than pairs
    (1, 130, 4, 8, 136, 1, 136),         # five
    (2, 224, 11, 3, 192, 1, 96),         # seven, identity replicated twice
    (1, 256, 13, 13, 256, 2, 64),        # stride 2, identity replicated four times
    (25, 64, 53, 53, 40, 1, 40),         # 64 channels a wave, the second word of the tile partial
    (12, 160, 53, 53, 128, 1, 128),      # two waves along the channels
]


@pytest.mark.parametrize("half", REAL_PARAMS, ids=REAL_IDS)
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_module_stream(shape, half):
    dev = gpu_device()
    n, c, h, w, o, stride, idc = shape
    seed = 71000 + 11 * c + h
    x, wt = W.pm1(seed, (n, c, h, w), 0.5), W.pm1(seed + 1, (o, c, 1, 1))
    y = oracle.conv2d_pm1(x, wt, stride, 0)
    m, cwo = y.size // o, (o + 31) // 32
    g, b = W.uniform_f32(seed + 2, (o,), -0.3, 0.3), W.uniform_f32(seed + 3, (o,), -3.0, 3.0)
    alpha, nxt = W.uniform_f32(seed + 4, (o,), -0.5, 1.5), W.uniform_f32(seed + 5, (o,), -5.0, 5.0)
    ident = real_store(W.uniform_f32(seed + 6, (m, idc), -9.0, 9.0), half)
    id32 = np.tile(real_values(ident, half), (1, o // idc))
    _, r32 = oracle.module_epilogue(y, g, b, id32.reshape(y.shape), alpha)
    want = real_store(r32.reshape(m, o), half)
    bits = oracle.pack_channels(oracle.sign_bias_f32(real_values(want, half).reshape(m, o, 1), nxt).reshape(m, o, 1))[:, 0, :]
    esz = np.dtype(real_np_dtype(half)).itemsize
    d = B.conv_desc(n, c, h, w, o, 1, stride, 0)
    xp = up(i32(oracle.pack_channels(x.reshape(n, c, -1))), dev)
    wp = up(i32(oracle.pack_channels(wt.reshape(o, c, 1))), dev)
    idb = Guarded.of_bytes(m * idc * esz, dev)
    idb.put(ident)
    for in_place in ((False, True) if idc == o else (False,)):
        r, xn = idb if in_place else Guarded.of_bytes(m * o * esz, dev), Guarded(m * cwo, dev)
        B.check(B.bcnn_conv2d_binary_module(d, xp, wp, up(g, dev), up(b, dev), idb.ptr, up(alpha, dev), up(nxt, dev),
                                            real_code(half), r.ptr, xn.ptr, identity_channels=idc), "module")
        assert np.array_equal(r.get(real_np_dtype(half), m * o).reshape(m, o), want)
        assert np.array_equal(xn.get(np.uint32).reshape(m, cwo), bits)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16], ids=str)
@pytest.mark.parametrize("c_out", [8, 64, 136])
def test_special_values(c_out, dtype):
    """Zeros of both signs, infinities, NaN, the types' largest and subnormal values in identity and parameters: the same
    stream and the same bits as the vector-ALU kernel's (which has the oracle's plain comparison), NaN in the same places."""
    gpu_device()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(72000 + c_out)
    m, c = 999, 96
    inf, nan, top = float("inf"), float("nan"), torch.finfo(dtype).max
    odd = torch.tensor([0.0, -0.0, inf, -inf, nan, top, -top, 6e-8, -6e-8, 1e-45, -1e-45, 70000.0, -70000.0, 1.5, -1.5], device="cuda")

    def pick(shape):
        plain = torch.rand(shape, generator=gen, device="cuda") * 20 - 10
        at = torch.randint(0, 2 * len(odd), shape, generator=gen, device="cuda")
        return torch.where(at < len(odd), odd[at % len(odd)], plain)

    x = torch.randint(-2 ** 31, 2 ** 31 - 1, (m, c // 32), generator=gen, device="cuda").to(torch.int32)
    wt = torch.randint(-2 ** 31, 2 ** 31 - 1, (c_out, c // 32), generator=gen, device="cuda").to(torch.int32)
    ident = pick((m, c_out)).to(dtype)
    ident[: m // 2] = -0.0                              # sums that are zeros of either sign, too
    g, b, slope, nxt = (pick((c_out,)) for _ in range(4))
    g[::2], b[::4], nxt[::3] = 0.0, -0.0, -0.0
    slope[::5] = 0.0
    d = B.conv_desc(1, c, m, 1, c_out, 1, 1, 0)
    code = {torch.float32: B.BCNN_F32, torch.float16: B.BCNN_F16, torch.bfloat16: B.BCNN_BF16}[dtype]
    got = []
    for variant in (B.BCNN_VARIANT_AUTO, B.BCNN_VARIANT_VALU):
        r = torch.empty((m, c_out), dtype=dtype, device="cuda")
        xn = torch.empty((m, (c_out + 31) // 32), dtype=torch.int32, device="cuda")
        B.check(B.bcnn_conv2d_binary_module(d, x, wt, g, b, ident, slope, nxt, code, r, xn, variant), "module")
        got.append((r, xn))
    (r0, x0), (r1, x1) = got
    raw = torch.int32 if dtype == torch.float32 else torch.int16
    none = torch.isnan(r1)
    assert torch.equal(torch.isnan(r0), none) and none.any() and (~none).any()
    assert torch.equal(r0.view(raw)[~none], r1.view(raw)[~none])
    assert torch.equal(x0, x1)
