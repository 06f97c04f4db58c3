"""Binarise + pack of channel-last rows and 2x2 to 4x4 pooling of 16-bit maps, against the oracle: channel counts around
the eight of a thread and the 32 of a word (ragged ones too), rows around a block's passes, replicated channels, sources
at 4-byte alignment, special values."""
import numpy as np
import pytest
import torch

import oracle
from paper_2010_00704_amd import binding as B
from paper_2010_00704_amd import workloads as W
from gpu_helpers import Guarded, gpu_device, real_code, real_np_dtype, real_store, real_values, up

pytestmark = pytest.mark.gpu

ROWS = [
    # rows, source channels, replication
    (1, 8, 1), (65, 2, 1), (257, 30, 1), (63, 32, 3), (1000, 44, 1), (129, 100, 1), (4097, 128, 2), (33, 264, 1),
    (5, 2048, 1), (7, 512, 4), (3, 1000, 2), (2, 2052, 1), (50, 36, 2),
]


def values(seed, shape):
    """Values on a coarse grid (exact zeros after the bias are common), with zeros of both signs, infinities and NaN."""
    v = W.uniform_f32(seed, shape, -4.0, 4.0, steps=32)
    f = v.reshape(-1)
    for k, s in enumerate([0.0, -0.0, np.inf, -np.inf, np.nan]):
        f[k::97] = s
    return v


@pytest.mark.parametrize("kind", [False, True, "bf16", "i8"], ids=["f32", "f16", "bf16", "i8"])
@pytest.mark.parametrize("shape", ROWS, ids=lambda s: "x".join(map(str, s)))
def test_pack_rows(shape, kind):
    dev = gpu_device()
    m, c, rep = shape
    if kind == "i8":
        stored = (W.raw_u64(m + c, 0, m * c) >> np.uint64(40)).astype(np.int64).astype(np.int8).reshape(m, c)
        v32, code = stored.astype(np.float32), B.BCNN_I8
    else:
        stored = real_store(values(90 + c, (m, c)), kind)
        v32, code = real_values(stored, kind), real_code(kind)
    raw = stored.view(np.uint8).reshape(-1)
    buf = torch.zeros(raw.size + 16, dtype=torch.uint8, device=dev)
    off = 4 if m % 2 else 0
    buf[off:off + raw.size] = torch.from_numpy(raw.copy()).to(dev)
    cr = rep * c
    bias = W.uniform_f32(91 + c, (cr,), -2.0, 2.0, steps=16)
    out = Guarded(m * ((cr + 31) // 32), dev)
    B.check(B.bcnn_pack_bias_replicated(buf.data_ptr() + off, code, m, c, 1, rep, up(bias, dev), out.ptr), "replicated")
    s = oracle.sign_bias_f32(np.tile(v32, (1, rep)).reshape(m, cr, 1), bias)
    assert np.array_equal(out.get(np.uint32).reshape(m, -1), oracle.pack_channels(s.reshape(m, cr, 1))[:, 0, :])
    if rep == 1:
        out = Guarded(m * ((c + 31) // 32), dev)
        B.check(B.bcnn_pack(buf.data_ptr() + off, code, m, c, 1, out.ptr), "pack")
        s = oracle.sign_f32(v32.reshape(m, c, 1))
        assert np.array_equal(out.get(np.uint32).reshape(m, -1), oracle.pack_channels(s.reshape(m, c, 1))[:, 0, :])


POOLS = [
    # n, h, w, channels, window
    (1, 2, 2, 8, 2), (2, 9, 7, 40, 2), (3, 31, 30, 64, 2), (1, 7, 65, 200, 2), (2, 10, 11, 32, 3), (1, 13, 9, 2048, 3),
    (5, 8, 9, 72, 4), (1, 4, 4, 1000, 4), (29, 146, 147, 16, 3), (17, 255, 256, 8, 4), (16, 255, 256, 8, 4),
]


@pytest.mark.parametrize("half", [True, "bf16"], ids=["f16", "bf16"])
@pytest.mark.parametrize("shape", POOLS, ids=lambda s: "x".join(map(str, s)))
def test_pool_eight_channels(shape, half):
    dev = gpu_device()
    n, h, w, c, s = shape
    stored = real_store(W.uniform_f32(95 + c + h, (n, h, w, c), -30.0, 30.0), half)
    bias = W.uniform_f32(96 + c, (c,), -5.0, 5.0)
    _, p32 = oracle.avgpool_nhwc(real_values(stored, half).reshape(n, h, w, c), s)
    m = p32.size // c
    want = real_store(p32.reshape(m, c), half)
    bits = oracle.pack_channels(oracle.sign_bias_f32(real_values(want, half).reshape(m, c, 1), bias).reshape(m, c, 1))[:, 0, :]
    src = torch.from_numpy(np.ascontiguousarray(stored).view(np.uint8).reshape(-1)).to(dev)
    for with_pooled, with_bits in ((True, True), (True, False), (False, True)):
        pooled, xp = Guarded.of_bytes(m * c * 2, dev), Guarded(m * ((c + 31) // 32), dev)
        B.check(B.bcnn_avgpool_bias_sign_pack(src, real_code(half), n, h, w, c, s, up(bias, dev),
                                              pooled.ptr if with_pooled else None, xp.ptr if with_bits else None), "pool")
        if with_pooled:
            assert np.array_equal(pooled.get(real_np_dtype(half), m * c).reshape(m, c), want)
        if with_bits:
            assert np.array_equal(xp.get(np.uint32).reshape(m, -1), bits)
