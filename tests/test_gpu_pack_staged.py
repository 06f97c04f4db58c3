"""Binarise + pack of [outer][C][inner] sources whose rows go through LDS (launches of 2048 groups of 64 channels and more), against the
oracle: rows of whole vectors, of whole dwords and of neither, around every number of vectors, channel counts around 32 and 64,
replicated channels, sources at 4-byte alignment, special values."""
import numpy as np
import pytest
import torch

import oracle
from paper_2010_00704_amd import binding as B
from paper_2010_00704_amd import workloads as W
from gpu_helpers import Guarded, gpu_device, real_code, real_store, real_values, up

pytestmark = pytest.mark.gpu

SHAPES = [
    # outer, source channels, inner, replication (channels in all: replication times as many)
    (2048, 64, 5, 1), (1025, 128, 9, 1), (1025, 66, 9, 1), (2049, 36, 16, 1), (700, 160, 17, 1), (1024, 65, 25, 1), (1024, 68, 25, 1), (690, 64, 28, 3),
    (690, 192, 33, 1), (2050, 64, 30, 1), (700, 192, 23, 1), (690, 190, 44, 1), (512, 256, 49, 1), (515, 252, 49, 1), (345, 128, 49, 3), (683, 130, 52, 1), (1024, 96, 56, 1), (512, 252, 63, 1), (2051, 60, 64, 1),
]


def offset(n):
    """Where in its allocation a source starts: sources are at 4-byte alignment."""
    return 4 if n % 2 else 0


def element_size(dtype):
    return torch.empty(0, dtype=dtype).element_size()


def images(size, c, inner):
    """An even number of them, a little more than 300 MB."""
    return (300 << 20) // (c * inner * size) // 2 * 2


@pytest.mark.parametrize("kind", [False, True, "bf16", "i8"], ids=["f32", "f16", "bf16", "i8"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pack_planes_through_lds(shape, kind):
    dev = gpu_device()
    n, c, inner, rep = shape
    if kind == "i8":
        stored = (W.raw_u64(n + c, 0, n * c * inner) >> np.uint64(40)).astype(np.int64).astype(np.int8).reshape(n, c, inner)
        v32, code = stored.astype(np.float32), B.BCNN_I8
    else:
        v = W.uniform_f32(180 + c + inner, (n, c, inner), -4.0, 4.0, steps=32)
        for k, s in enumerate([0.0, -0.0, np.inf, -np.inf, np.nan]):
            v.reshape(-1)[k::97] = s
        stored = real_store(v, kind)
        v32, code = real_values(stored, kind).reshape(n, c, inner), real_code(kind)
    raw = np.ascontiguousarray(stored).view(np.uint8).reshape(-1)
    off = offset(n)
    buf = torch.zeros(raw.size + 16, dtype=torch.uint8, device=dev)
    buf[off:off + raw.size] = torch.from_numpy(raw.copy()).to(dev)
    cr = rep * c
    bias = W.uniform_f32(181 + c, (cr,), -2.0, 2.0, steps=16)
    out = Guarded(n * inner * ((cr + 31) // 32), dev)
    B.check(B.bcnn_pack_bias_replicated(buf.data_ptr() + off, code, n, c, inner, rep, up(bias, dev), out.ptr), "replicated")
    s = oracle.sign_bias_f32(np.tile(v32, (1, rep, 1)), bias)
    assert np.array_equal(out.get(np.uint32).reshape(n, inner, -1), oracle.pack_channels(s))
    if rep == 1:
        out = Guarded(n * inner * ((c + 31) // 32), dev)
        B.check(B.bcnn_pack(buf.data_ptr() + off, code, n, c, inner, out.ptr), "pack")
        assert np.array_equal(out.get(np.uint32).reshape(n, inner, -1), oracle.pack_channels(oracle.sign_f32(v32)))


BEYOND_THE_CACHE = [
    # element type, channels, inner: rows of whole vectors, of whole dwords and of neither
    (torch.bfloat16, 256, 56), (torch.float16, 200, 34), (torch.float16, 130, 25), (torch.int8, 96, 64), (torch.int8, 100, 49), (torch.float32, 64, 28), (torch.float32, 65, 9),
]


@pytest.mark.parametrize("dtype,c,inner", BEYOND_THE_CACHE, ids=lambda v: str(v).replace("torch.", ""))
def test_pack_planes_beyond_the_cache(dtype, c, inner):
    """Sources of more than 288 MB are loaded past the caches' lines; their parts, each below that, are not."""
    dev = gpu_device()
    code = {torch.float32: B.BCNN_F32, torch.float16: B.BCNN_F16, torch.bfloat16: B.BCNN_BF16, torch.int8: B.BCNN_I8}[dtype]
    n = images(element_size(dtype), c, inner)
    g = torch.Generator(device=dev)
    g.manual_seed(c + inner)
    x = torch.randint(-100, 101, (n, c, inner), generator=g, device=dev, dtype=torch.int8).to(dtype)
    bias = torch.randint(-3, 4, (c,), generator=g, device=dev).float()
    words = n * inner * ((c + 31) // 32)
    whole, parts = Guarded(words, dev), Guarded(words, dev)
    B.check(B.bcnn_pack_bias(x.data_ptr(), code, n, c, inner, bias, whole.ptr), "whole")
    for k in range(2):
        B.check(B.bcnn_pack_bias(x[k * n // 2].data_ptr(), code, n // 2, c, inner, bias, parts.ptr + 4 * k * (words // 2)), "part")
    assert np.array_equal(whole.get(), parts.get())
    assert len(np.unique(whole.get()[:4096])) > 100
