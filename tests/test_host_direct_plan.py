"""Host logic: which tile of the direct kernel a call takes (csrc/direct_plan.h), on measured calls, and that the GPU test of
the tiles reaches every one of them.  Compiled for the host with g++ and run here; no GPU involved."""
import os
import subprocess

import pytest

import test_gpu_direct_tiles as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("direct_plan") / "direct_plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_00704_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "direct_plan_check.cpp"), "-o", exe], check=True)
    return exe


def test_measured_calls_go_to_the_faster_kernel(checker):
    out = subprocess.run([checker], stdout=subprocess.PIPE, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    assert "mismatches: 0" in out.stdout


def choices(checker, mode, calls):
    lines = "\n".join(" ".join(str(int(v)) for v in c) for c in calls)
    out = subprocess.run([checker, mode], input=lines, stdout=subprocess.PIPE, text=True, timeout=300, check=True)
    return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]


def test_every_tile_and_walk_is_reached_on_the_gpu(checker):
    """The GPU test's shapes take the tiles and walks that it lists, and the list is whole: whatever AUTO chooses over a grid of
    calls that no rule gives to another kernel is in it."""
    listed = {(kind, tile, walk) for kind, tile, walk, _ in G.CONVS}
    calls = [(n * h * w, o, (c + 31) // 32, k, kind, False) for kind, _, _, (n, c, h, w, o, k) in G.CONVS]
    assert choices(checker, "conv", calls) == [(tile, walk) for _, tile, walk, _ in G.CONVS]
    grid = [(m, o, cw, ks, kind, False) for m in (1, 196, 784, 3136, 12544, 50176, 200704) for o in (16, 64, 100, 256, 512)
            for cw in (1, 2, 3, 4, 5, 8, 9, 16, 32) for ks in (1, 3) for kind in (G.BITS, G.SUMS, G.MODULE)]
    assert {(c[4], tile, walk) for c, (tile, walk) in zip(grid, choices(checker, "conv", grid))} <= listed


def test_every_branch_tile_is_reached_on_the_gpu(checker):
    def key(out):
        return out.startswith("module"), out == "module_f16"

    calls = [(n * h * w, o, (c + 31) // 32, taps, *key(out)) for out, _, (n, c, h, w, o, taps) in G.BRANCHES]
    assert [tile for tile, _ in choices(checker, "branches", calls)] == [tile for _, tile, _ in G.BRANCHES]
    listed = {(key(out), tile) for out, tile, _ in G.BRANCHES}
    grid = [(m, o, cw, p, *key(out)) for m in (1, 784, 12544, 50176, 200704) for o in (32, 100, 256, 512) for cw in (1, 3, 7, 8, 16, 32)
            for p in (1, 2, 9, 16) for out in G.OUTS]
    assert {((bool(c[4]), bool(c[5])), tile) for c, (tile, _) in zip(grid, choices(checker, "branches", grid))} <= listed
