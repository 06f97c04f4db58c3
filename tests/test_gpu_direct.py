"""The matrix-core convolution without LDS staging, through the calls that AUTO routes to it, against the oracle:
channel counts around every unit of its K walk (words per tap 1 to 12, with and without tail bits), pixel and channel
counts around its 32 x 32 blocks and its 128-pixel workgroups, strides, borders, operands at 4-byte alignment.  (Every
tile with every walk: test_gpu_direct_tiles.py.)"""
import numpy as np
import pytest
import torch

import oracle
from paper_2010_00704_amd import binding as B
from paper_2010_00704_amd import workloads as W
from gpu_helpers import Guarded, gpu_device, i32, real_code, real_np_dtype, real_store, real_values, up

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, c_in, h, w, c_out, k, stride, pad
    (1, 1, 1, 1, 1, 1, 1, 0),            # one word, one pixel
    (1, 31, 5, 7, 33, 3, 1, 1),          # one word per tap: nine words, the last unit holds one
    (2, 64, 9, 7, 31, 3, 2, 1),          # two words per tap, odd map under stride 2
    (1, 96, 6, 6, 64, 3, 1, 0),          # three words per tap, no padding
    (3, 128, 8, 4, 65, 3, 1, 1),         # four: whole units
    (1, 129, 7, 7, 32, 3, 1, 1),         # five: tail unit shares three words
    (1, 190, 5, 9, 40, 3, 2, 1),         # six
    (2, 224, 4, 4, 96, 3, 1, 1),         # seven: shares one
    (1, 288, 6, 5, 130, 1, 2, 0),        # 1x1, nine words, stride 2
    (2, 360, 7, 7, 100, 3, 1, 1),        # twelve words with tail bits
    (1, 1024, 7, 7, 256, 3, 1, 1),       # K split over four waves, single image
    (40, 544, 15, 15, 250, 3, 1, 1),     # 2 x 2 blocks per wave, K split, 17 words per tap
    (40, 40, 28, 28, 72, 1, 1, 0),       # one block, four waves side by side, ragged last pixel block
    (61, 70, 29, 29, 161, 3, 1, 1),      # 2 x 1 blocks, four waves side by side, ragged on both sides
]


@pytest.fixture(scope="module")
def dev():
    return gpu_device()


def pack_x(s):
    n, c = s.shape[:2]
    return i32(oracle.pack_channels(s.reshape(n, c, -1)))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "word_aligned"])
def test_direct(dev, shape, offset):
    n, c, h, w, o, k, stride, pad = shape
    seed = 52000 + c * 7 + h
    x, wt = W.pm1(seed, (n, c, h, w), 0.45), W.pm1(seed + 1, (o, c, k, k))
    y = oracle.conv2d_pm1(x, wt, stride, pad)
    thr = (np.median(y, axis=(0, 1, 2)).astype(np.int32) if y.size < 1 << 22 else W.thresholds(seed + 2, o, 16))
    m, cwo = y.size // o, (o + 31) // 32

    def place(a):                        # `offset` words past an allocation's start
        t = torch.zeros(a.size + 4, dtype=torch.int32, device=dev)
        t[offset:offset + a.size] = torch.from_numpy(a.reshape(-1)).to(dev)
        return t, t.data_ptr() + 4 * offset
    xt, xp = place(pack_x(x))
    wtt, wp = place(i32(oracle.pack_channels(wt.reshape(o, c, k * k))))
    d = B.conv_desc(n, c, h, w, o, k, stride, pad)
    sums, bits = Guarded(m * o, dev), Guarded(m * cwo, dev)
    B.check(B.bcnn_conv2d_binary(d, xp, wp, sums.ptr), "sums")
    B.check(B.bcnn_conv2d_binary_sign_pack(d, xp, wp, up(thr, dev), bits.ptr), "bits")
    assert np.array_equal(sums.get(np.int32).reshape(m, o), y.reshape(m, o))
    s = oracle.threshold_sign(y, thr).reshape(m, o, 1)
    assert np.array_equal(bits.get(np.uint32).reshape(m, cwo), oracle.pack_channels(s)[:, 0, :])

    # the module epilogue on the same sums: every part present, then without identity, slope and next bias
    half = [False, True, "bf16"][(c + o) % 3]
    g, b = W.uniform_f32(seed + 3, (o,), -0.3, 0.3), W.uniform_f32(seed + 4, (o,), -3.0, 3.0)
    alpha, nxt = W.uniform_f32(seed + 5, (o,), 0.05, 0.5), W.uniform_f32(seed + 6, (o,), -5.0, 5.0)
    ident = real_store(W.uniform_f32(seed + 7, (m, o), -9.0, 9.0), half)
    esz = np.dtype(real_np_dtype(half)).itemsize
    for full in (True, False):
        r, xn = Guarded.of_bytes(m * o * esz, dev), Guarded(m * cwo, dev)
        B.check(B.bcnn_conv2d_binary_module(
            d, xp, wp, up(g, dev), up(b, dev), up_bytes(ident, dev) if full else None, up(alpha, dev) if full else None,
            up(nxt, dev) if full else None, real_code(half), r.ptr, xn.ptr), "module")
        id32 = real_values(ident, half).reshape(y.shape) if full else None
        _, r32 = oracle.module_epilogue(y, g, b, id32, alpha if full else None)
        want = real_store(r32.reshape(m, o), half)
        sb = oracle.sign_bias_f32(real_values(want, half).reshape(m, o, 1), nxt if full else np.zeros(o, np.float32))
        assert np.array_equal(r.get(real_np_dtype(half), m * o).reshape(m, o), want)
        assert np.array_equal(xn.get(np.uint32).reshape(m, cwo), oracle.pack_channels(sb.reshape(m, o, 1))[:, 0, :])
    del xt, wtt


def up_bytes(a, dev):
    """Any real type as raw bytes on the device."""
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1)).to(dev)


PARTS = [(True, True, False), (True, False, True), (False, True, True), (False, True, False), (False, False, True)]


@pytest.mark.parametrize("half", [False, True, "bf16"], ids=["f32", "f16", "bf16"])
@pytest.mark.parametrize("parts", PARTS, ids=lambda p: "".join(n for n, on in zip(("id", "r", "x"), p) if on))
@pytest.mark.parametrize("shape", [(2, 130, 7, 6, 64, 3, 1, 1), (3, 64, 9, 9, 36, 1, 2, 0), (40, 96, 28, 28, 72, 1, 1, 0)],
                         ids=lambda s: "x".join(map(str, s)))
def test_module_without_some_parts(dev, shape, parts, half):
    """Identity, real stream or next packing missing where channels come in whole fours; some channels give -0 or +0, which
    a missing identity leaves as it is."""
    n, c, h, w, o, k, stride, pad = shape
    has_id, has_r, has_x = parts
    seed = 53000 + c + 7 * o
    x, wt = W.pm1(seed, (n, c, h, w), 0.45), W.pm1(seed + 1, (o, c, k, k))
    y = oracle.conv2d_pm1(x, wt, stride, pad)
    m, cwo = y.size // o, (o + 31) // 32
    g, b = W.uniform_f32(seed + 3, (o,), -0.3, 0.3), W.uniform_f32(seed + 4, (o,), -3.0, 3.0)
    g[::5], b[::5] = 0.0, -0.0
    alpha, nxt = W.uniform_f32(seed + 5, (o,), 0.05, 0.5), W.uniform_f32(seed + 6, (o,), -5.0, 5.0)
    ident = real_store(W.uniform_f32(seed + 7, (m, o), -9.0, 9.0), half)
    esz = np.dtype(real_np_dtype(half)).itemsize
    d = B.conv_desc(n, c, h, w, o, k, stride, pad)
    r, xn = Guarded.of_bytes(m * o * esz, dev), Guarded(m * cwo, dev)
    B.check(B.bcnn_conv2d_binary_module(
        d, up(pack_x(x), dev), up(i32(oracle.pack_channels(wt.reshape(o, c, k * k))), dev), up(g, dev), up(b, dev),
        up_bytes(ident, dev) if has_id else None, up(alpha, dev), up(nxt, dev), real_code(half), r.ptr if has_r else None,
        xn.ptr if has_x else None), "module")
    _, r32 = oracle.module_epilogue(y, g, b, real_values(ident, half).reshape(y.shape) if has_id else None, alpha)
    want = real_store(r32.reshape(m, o), half)
    if has_r:
        assert np.array_equal(r.get(real_np_dtype(half), m * o).reshape(m, o).view(np.uint8), want.view(np.uint8))
    else:
        assert np.all(r.get(np.uint32) == 0x5A5A5A5A)
    if has_x:
        sb = oracle.sign_bias_f32(real_values(want, half).reshape(m, o, 1), nxt)
        assert np.array_equal(xn.get(np.uint32).reshape(m, cwo), oracle.pack_channels(sb.reshape(m, o, 1))[:, 0, :])
    else:
        assert np.all(xn.get(np.uint32) == 0x5A5A5A5A)
