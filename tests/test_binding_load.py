"""The binding where its marshalling extension does not load: calls take ctypes, under the same rules."""
import importlib.machinery
import importlib.util
import subprocess
import sys

import pytest
import torch

from paper_2010_00704_amd import binding as B
from paper_2010_00704_amd import build
from test_binding_marshal import test_taken_and_refused as taken_and_refused

CASES = next(m for m in taken_and_refused.pytestmark if m.name == "parametrize").args[1]

WITHOUT = """
import sys, warnings
sys.modules["paper_2010_00704_amd._marshal"] = None          # an import of it raises ImportError
from paper_2010_00704_amd import binding as B
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    assert B.bcnn_pack(None, 0, 1, 1, 1, 64, 0) == B.BCNN_ERR_INVALID_ARG
    assert B.bcnn_pack(None, 0, 1, 1, 1, 64, 0) == B.BCNN_ERR_INVALID_ARG
assert [w.category for w in seen if "_marshal.so" in str(w.message)] == [RuntimeWarning], seen
"""


def test_loads_without_the_extension():
    subprocess.run([sys.executable, "-c", WITHOUT], cwd=build._ROOT, check=True, timeout=300)


def test_extension_refuses_another_torch(tmp_path):
    path = build.build_marshal(str(tmp_path / "_marshal.so"), torch_version="0.1")
    loader = importlib.machinery.ExtensionFileLoader("_marshal", path)
    with pytest.raises(ImportError, match="torch 0.1"):
        importlib.util.module_from_spec(importlib.util.spec_from_loader("_marshal", loader))


@pytest.fixture
def by_ctypes(monkeypatch):
    B.lib()
    monkeypatch.setattr(B, "_marshal", B._Ctypes)


@pytest.mark.parametrize("call,want", CASES)
def test_taken_and_refused(by_ctypes, call, want):
    taken_and_refused(call, want)


@pytest.mark.gpu
@pytest.mark.parametrize("face", ["extension", "ctypes"])
def test_same_results(face, monkeypatch):
    """Every marshalled call on small tensors, against itself through the other face."""
    assert torch.cuda.is_available()
    B.lib()
    n, c, h, w, o = 2, 40, 9, 7, 36
    m, words = n * h * w, 2
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def real(*shape):
        return torch.rand(shape, generator=gen, device="cuda") * 2 - 1

    src, weights, bias, scale, slope, ident = real(n, c, h * w), real(o, c, 9), real(c), real(9, o), real(o), real(m, o)
    thr = (real(o) * 20).to(torch.int32)
    desc = B.conv_desc(n, c, h, w, o, 3, 1, 1)

    def run():
        def ints(*shape):
            return torch.zeros(shape, dtype=torch.int32, device="cuda")

        def floats(*shape):
            return torch.zeros(shape, device="cuda")

        x, xb, xr, wt, pad = ints(m, words), ints(m, words), ints(m, 3), ints(o * 9, words), ints(9, words)
        y, bits, var, again = ints(m, o), ints(m, words), ints(m, words), ints(m, words)
        r, xn, z, zb, zr, zx = floats(m, o), ints(m, words), floats(m, o), ints(m, words), floats(m, o), ints(m, words)
        pooled, pb = floats(n * 4 * 3, o), ints(n * 4 * 3, words)
        for status in (
                B.bcnn_pack(src, B.BCNN_F32, n, c, h * w, x), B.bcnn_pack(weights, B.BCNN_F32, o, c, 9, wt),
                B.bcnn_pack_bias(src, B.BCNN_F32, n, c, h * w, bias, xb),
                B.bcnn_pack_bias_replicated(src, B.BCNN_F32, n, c, h * w, 2, torch.cat([bias, -bias]), xr),
                B.bcnn_conv2d_binary(desc, x, wt, y), B.bcnn_conv2d_binary_sign_pack(desc, x, wt, thr, bits),
                B.bcnn_conv2d_binary_variant(desc, xb, wt, thr, var, B.BCNN_VARIANT_AUTO),
                B.bcnn_threshold_sign_pack(y, thr, m, o, again),
                B.bcnn_conv2d_binary_module(desc, x, wt, slope, slope, ident, slope, None, B.BCNN_F32, r, xn),
                B.bcnn_conv2d_binary_branches(desc, 9, x, 0, wt, pad, B.BCNN_PAD_WORDS, scale, slope, z),
                B.bcnn_conv2d_binary_branches_sign_pack(desc, 9, x, 0, wt, None, B.BCNN_PAD_ZERO, scale, slope, zb),
                B.bcnn_conv2d_binary_branches_module(desc, 9, x, 0, wt, pad, B.BCNN_PAD_WORDS, scale, slope, ident, slope, slope,
                                                     B.BCNN_F32, zr, zx),
                B.bcnn_avgpool_bias_sign_pack(ident, B.BCNN_F32, n, h, w, o, 2, slope, pooled, pb)):
            B.check(status)
        torch.cuda.synchronize()
        return [x, xb, xr, wt, y, bits, var, again, r, xn, z, zb, zr, zx, pooled, pb]

    want = run()
    if face == "ctypes":
        monkeypatch.setattr(B, "_marshal", B._Ctypes)
    got = run()
    assert all(torch.equal(a, b) for a, b in zip(want, got))
    assert all(t.any() for t in got)
    assert torch.equal(got[5], got[7])                        # bits of the sums' thresholds, both ways
