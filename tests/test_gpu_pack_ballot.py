"""Binarise + pack of [outer][C][inner] sources with lanes along the channels, against the oracle: row lengths around a
vector, a wave's 64 positions and a cache line, rows that start at any byte, channel counts around 32 and 64, replicated
channels, images that are no whole number of dwords (another kernel), sources at 4-byte alignment, special values."""
import numpy as np
import pytest
import torch

import oracle
from paper_2010_00704_amd import binding as B
from paper_2010_00704_amd import workloads as W
from gpu_helpers import Guarded, gpu_device, real_code, real_store, real_values, up

pytestmark = pytest.mark.gpu

SHAPES = [
    # outer, source channels, inner, replication
    (1, 2, 2, 1), (3, 33, 3, 1), (70, 64, 9, 1), (2, 65, 16, 2), (5, 130, 33, 1), (37, 200, 49, 1), (2, 1024, 49, 1),
    (3, 96, 56, 3), (2, 64, 57, 1), (9, 31, 64, 1), (1, 66, 65, 1), (4, 192, 127, 1), (3, 193, 128, 1), (2, 320, 625, 1),
    (12, 288, 784, 1), (70, 256, 512, 1), (90, 64, 441, 1),
]


@pytest.mark.parametrize("kind", [False, True, "bf16", "i8"], ids=["f32", "f16", "bf16", "i8"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pack_planes(shape, kind):
    dev = gpu_device()
    n, c, inner, rep = shape
    if kind == "i8":
        stored = (W.raw_u64(n + c, 0, n * c * inner) >> np.uint64(40)).astype(np.int64).astype(np.int8).reshape(n, c, inner)
        v32, code = stored.astype(np.float32), B.BCNN_I8
    else:
        v = W.uniform_f32(80 + c + inner, (n, c, inner), -4.0, 4.0, steps=32)
        for k, s in enumerate([0.0, -0.0, np.inf, -np.inf, np.nan]):
            v.reshape(-1)[k::97] = s
        stored = real_store(v, kind)
        v32, code = real_values(stored, kind).reshape(n, c, inner), real_code(kind)
    raw = np.ascontiguousarray(stored).view(np.uint8).reshape(-1)
    off = 4 if n % 2 else 0
    buf = torch.zeros(raw.size + 16, dtype=torch.uint8, device=dev)
    buf[off:off + raw.size] = torch.from_numpy(raw.copy()).to(dev)
    cr = rep * c
    bias = W.uniform_f32(81 + c, (cr,), -2.0, 2.0, steps=16)
    out = Guarded(n * inner * ((cr + 31) // 32), dev)
    B.check(B.bcnn_pack_bias_replicated(buf.data_ptr() + off, code, n, c, inner, rep, up(bias, dev), out.ptr), "replicated")
    s = oracle.sign_bias_f32(np.tile(v32, (1, rep, 1)), bias)
    assert np.array_equal(out.get(np.uint32).reshape(n, inner, -1), oracle.pack_channels(s))
    if rep == 1:
        out = Guarded(n * inner * ((c + 31) // 32), dev)
        B.check(B.bcnn_pack(buf.data_ptr() + off, code, n, c, inner, out.ptr), "pack")
        assert np.array_equal(out.get(np.uint32).reshape(n, inner, -1), oracle.pack_channels(oracle.sign_f32(v32)))


@pytest.mark.parametrize("inner", [2, 5])
def test_more_images_than_a_launch_has_workgroups(inner):
    """2^24 images of two channels: a launch holds fewer than 2^32 threads, so not a workgroup of 256 per image."""
    dev = gpu_device()
    n = 1 << 24
    src = torch.randint(-100, 101, (n, 2, inner), dtype=torch.int8, device=dev)
    out = torch.full((n, inner), 77, dtype=torch.int32, device=dev)
    B.check(B.bcnn_pack(src, B.BCNN_I8, n, 2, inner, out), "pack")
    on = src >= 0
    assert torch.equal(out, on[:, 0].int() + 2 * on[:, 1].int())
