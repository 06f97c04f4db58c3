"""Branch sums on the matrix cores without LDS staging, through the calls that AUTO routes to it, against the oracle:
words per lane half around a group of four (single words, whole groups, both), odd word counts, every pad mode, own and
shared tensors, ragged channels and pixels, operands at 4-byte alignment.  (Its tiles: test_gpu_direct_tiles.py.)"""
import random

import numpy as np
import pytest
import torch

import oracle
from paper_2010_00704_amd import binding as B
from paper_2010_00704_amd import workloads as W
from gpu_helpers import Guarded, gpu_device, i32, oracle_pack_nchw, oracle_pack_vectors, real_code, real_np_dtype, real_store, real_values, up

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, c_in, h, w, c_out, k, stride, branches, own tensors
    (1, 20, 4, 5, 33, 3, 1, 9, False),       # one word: the second half is empty
    (2, 64, 7, 7, 40, 3, 2, 9, True),        # two words, odd map under stride 2
    (1, 96, 9, 5, 32, 1, 1, 2, True),        # three
    (1, 230, 6, 6, 100, 3, 1, 9, False),     # eight: one whole group per half
    (2, 288, 5, 7, 64, 1, 1, 4, False),      # nine: a group and a single word, odd
    (1, 352, 7, 7, 65, 3, 1, 9, True),       # eleven
    (1, 512, 8, 8, 32, 1, 2, 16, True),      # two groups, the most branches that are kept in LDS
    # an odd count whose longer half is whole groups of four: the shorter half is a word short in its last group
    (1, 193, 4, 5, 33, 3, 1, 9, False),      # seven
    (2, 224, 7, 6, 40, 3, 2, 9, True),       # seven, odd map under stride 2
    (1, 224, 5, 9, 64, 1, 1, 3, True),       # seven, parallel branches
    (2, 224, 6, 4, 36, 1, 1, 2, False),      # seven, parallel branches of one tensor
    (1, 480, 6, 7, 70, 3, 1, 9, False),      # fifteen
    (1, 736, 5, 5, 32, 3, 1, 9, True),       # twenty-three
    (3, 992, 3, 4, 96, 1, 1, 4, True),       # thirty-one
    (60, 128, 28, 28, 96, 3, 1, 9, False),   # many workgroups, three channel blocks
    (20, 512, 28, 28, 288, 1, 1, 3, False),  # parallel branches, many workgroups
]


@pytest.fixture(scope="module")
def dev():
    return gpu_device()


def as_bytes(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1)).to(dev)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("mode", ["minus", "words", "zero"])
def test_branches_direct(dev, shape, mode):
    check(dev, shape, mode, 61000 + 13 * shape[1] + shape[2])


@pytest.mark.parametrize("shape", [(1, 226, 5, 6, 40, 3, 1, 9, False), (2, 250, 7, 4, 130, 3, 2, 9, True), (1, 500, 6, 5, 64, 1, 1, 4, True),
                                   (1, 737, 4, 4, 33, 3, 1, 9, False)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("mode", ["minus", "words", "zero"])
def test_staged_branches_with_a_partial_last_word(dev, shape, mode):
    """Channel counts short of whole 256-channel chunks on the kernel that stages its operands in LDS."""
    check(dev, shape, mode, 63000 + 13 * shape[1] + shape[2], B.BCNN_VARIANT_MFMA_FP4)


@pytest.mark.parametrize("seed", range(12))
def test_random_channel_counts(dev, seed):
    """Any channel count up to 1024 on small maps: every word count of a tap is as likely as another."""
    rng = random.Random(62000 + seed)
    for _ in range(4):
        k = rng.choice([1, 3])
        shape = (rng.randint(1, 3), rng.randint(1, 1024), rng.randint(3, 9), rng.randint(3, 9), rng.randint(32, 100), k,
                 rng.choice([1, 1, 2]), 9 if k == 3 else rng.randint(1, 5), rng.random() < 0.4)
        check(dev, shape, rng.choice(["minus", "words", "zero"]), rng.randrange(1 << 20))


def check(dev, shape, mode, seed, variant=B.BCNN_VARIANT_AUTO):
    n, c, h, w, o, k, stride, taps, own = shape
    pad = (k - 1) // 2
    xs = [W.pm1(seed + 20 + t, (n, c, h, w), 0.5) for t in range(taps if own else 1)]
    wt = W.pm1(seed, (o, c, taps))
    scale, bias = W.uniform_f32(seed + 1, (taps, o), -0.4, 0.4), W.uniform_f32(seed + 2, (o,), -3.0, 3.0)
    padv = {"minus": np.full((taps, c), -1, np.int8), "words": W.pm1(seed + 3, (taps, c)),
            "zero": np.zeros((taps, c), np.int8)}[mode]
    _, z = oracle.branches_pm1(np.stack(xs), padv, wt.reshape(o, c, k, k) if k == 3 else wt, scale, bias, stride, pad)
    m, cwo = z.size // o, (o + 31) // 32
    d = B.conv_desc(n, c, h, w, o, k, stride, pad)
    off = 1 if c % 3 == 0 else 0             # some operands a word past an allocation's start
    xw = np.concatenate([i32(oracle_pack_nchw(x)).reshape(-1) for x in xs])
    ww = i32(oracle.pack_channels(wt)).reshape(-1)
    xt, wtt = (torch.zeros(a.size + 4, dtype=torch.int32, device=dev) for a in (xw, ww))
    xt[off:off + xw.size] = torch.from_numpy(xw).to(dev)
    wtt[off:off + ww.size] = torch.from_numpy(ww).to(dev)
    pw = up(i32(oracle_pack_vectors(np.where(padv == 0, -1, padv).astype(np.int8))), dev)
    args = (d, taps, xt.data_ptr() + 4 * off, xw.size // taps if own else 0, wtt.data_ptr() + 4 * off,
            pw if mode == "words" else None, B.BCNN_PAD_ZERO if mode == "zero" else B.BCNN_PAD_WORDS, up(scale, dev), up(bias, dev))
    zf, bits = Guarded(m * o, dev), Guarded(m * cwo, dev)
    B.check(B.bcnn_conv2d_binary_branches(*args, zf.ptr, variant), "branches")
    B.check(B.bcnn_conv2d_binary_branches_sign_pack(*args, bits.ptr, variant), "sign_pack")
    assert np.array_equal(zf.get(np.float32).reshape(m, o), z.reshape(m, o))
    signs = np.where(z >= 0, 1, -1).astype(np.int8).reshape(m, o, 1)
    assert np.array_equal(bits.get(np.uint32).reshape(m, cwo), oracle.pack_channels(signs)[:, 0, :])

    # the module tail: every part present, then the real stream alone
    alpha, nxt = W.uniform_f32(seed + 5, (o,), 0.05, 0.5), W.uniform_f32(seed + 6, (o,), -5.0, 5.0)
    for half in (False, True):
        ident = real_store(W.uniform_f32(seed + 7, (m, o), -9.0, 9.0), half)
        esz = np.dtype(real_np_dtype(half)).itemsize
        for whole in (True, False):
            r, xn = Guarded.of_bytes(m * o * esz, dev), Guarded(m * cwo, dev)
            B.check(B.bcnn_conv2d_binary_branches_module(
                *args, as_bytes(ident, dev) if whole else None, up(alpha, dev) if whole else None,
                up(nxt, dev) if whole else None, real_code(half), r.ptr, xn.ptr, variant), "module")
            t = z.reshape(m, o).astype(np.float32)
            if whole:
                t = t + real_values(ident, half)
                t = np.where(t >= 0, t, alpha * t).astype(np.float32)
            want = real_store(t, half)
            sb = oracle.sign_bias_f32(real_values(want, half).reshape(m, o, 1), nxt if whole else np.zeros(o, np.float32))
            assert np.array_equal(r.get(real_np_dtype(half), m * o).reshape(m, o), want)
            assert np.array_equal(xn.get(np.uint32).reshape(m, cwo), oracle.pack_channels(sb.reshape(m, o, 1))[:, 0, :])
