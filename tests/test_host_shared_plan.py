"""Host logic: how the direct kernel's form with shared weights walks a tap's words and which calls take it
(csrc/shared_plan.h), and that its GPU test reaches every tile and width of loads.  Compiled for the host with g++."""
import os
import subprocess

import pytest

import test_gpu_shared_weights as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("shared_plan") / "shared_plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_00704_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "shared_plan_check.cpp"), "-o", exe], check=True)
    return exe


def test_every_word_is_walked_once(checker):
    out = subprocess.run([checker], stdout=subprocess.PIPE, text=True, timeout=300)
    assert out.returncode == 0, out.stdout


def choices(checker, calls, mode="calls"):
    lines = "\n".join(" ".join(str(int(v)) for v in c) for c in calls)
    out = subprocess.run([checker, mode], input=lines, stdout=subprocess.PIPE, text=True, timeout=300, check=True)
    return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]


def call(kind, n, c, h, w, o, k, stride):
    m = n * ((h - 1) // stride + 1) * ((w - 1) // stride + 1)
    return (m, o, (c + 31) // 32, k, min(kind, 3) if kind < 2 else 3, kind, 0)


def test_every_tile_and_width_is_reached_on_the_gpu(checker):
    got = choices(checker, [call(kind, *shape) for kind, _, _, shape in G.CONVS])
    assert got == [(tile, wide) for _, tile, wide, _ in G.CONVS]
    grid = [(m, o, cw, ks, kind if kind < 2 else 3, kind, 0) for m in (196, 784, 3136, 12544, 50176, 200704) for o in (16, 64, 100, 256, 512)
            for cw in (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 16, 18, 32) for ks in (1, 3) for kind in (G.BITS, G.SUMS, G.HALF, G.FLOAT)]
    listed = {(kind, tile, wide) for kind, tile, wide, _ in G.CONVS}
    reached = {(c[5], tile, wide) for c, (tile, wide) in zip(grid, choices(checker, grid)) if tile}
    assert reached <= listed, sorted(reached - listed)


def test_every_branch_form_is_reached_on_the_gpu(checker):
    def tail(out):
        return out.startswith("module"), out == "module_f16"

    calls = [(n * h * w, o, (c + 31) // 32, taps, *tail(out)) for _, _, _, out, (n, c, h, w, o, taps) in G.BRANCHES]
    assert choices(checker, calls, "branches") == [(form, tile, wide) for form, tile, wide, _, _ in G.BRANCHES]
    grid = [(m, o, cw, p, *tail(out)) for m in (49, 784, 12544, 50176, 200704) for o in (32, 100, 256, 512) for cw in (1, 3, 5, 8, 9, 16, 32)
            for p in (2, 3, 9, 16) for out in ("bits", "f32", "module_f32", "module_f16")]
    listed = {(form, tile, wide) for form, tile, wide, _, _ in G.BRANCHES if form == G.SHARED}
    assert {c for c in choices(checker, grid, "branches") if c[0] == G.SHARED} <= listed
