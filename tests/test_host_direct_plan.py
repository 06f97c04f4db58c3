"""Host logic: which tile of the direct kernel a call takes (csrc/direct_plan.h, and csrc/shared_plan.h, which decides after it), on
measured calls, and that the GPU test of the tiles reaches every one of them.  Compiled for the host with g++ and run here; no GPU involved."""
import os
import subprocess

import pytest

import test_gpu_direct_tiles as G
from test_host_shared_plan import checker as plan  # noqa: F401  (a fixture)
from test_host_shared_plan import choices as shared_choices

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


def test_every_tile_and_walk_is_reached_on_the_gpu(plan):
    """The GPU test's shapes take the tiles and walks that it lists, and the list is whole: whatever AUTO chooses over a grid of
    calls that no rule gives to another kernel is in it."""
    listed = {(kind, tile, walk) for kind, tile, walk, _ in G.CONVS}

    def line(kind, m, o, cw, ks, stride=1):
        return (m, o, cw, ks, stride, kind if kind < 2 else 3, kind, 0)

    calls = [line(kind, n * h * w, o, (c + 31) // 32, k) for kind, _, _, (n, c, h, w, o, k) in G.CONVS]
    assert choices(plan, calls) == [(0, (tile, walk)) for _, tile, walk, _ in G.CONVS]
    grid = [line(kind, m, o, cw, ks, stride) for m in (1, 196, 784, 3136, 12544, 50176, 200704) for o in (16, 64, 100, 256, 512)
            for cw in (1, 2, 3, 4, 5, 8, 9, 16, 32) for ks in (1, 3) for stride in (1, 2) for kind in (G.BITS, G.SUMS, G.HALF, G.FLOAT)]
    assert {(c[6], *tile) for c, (shared, tile) in zip(grid, choices(plan, grid)) if not shared} <= listed


def choices(plan, calls):
    """(tile of the form with shared weights or 0, (tile, walk) of the other choice) of each call"""
    return [(shared, (tile, walk)) for shared, _, tile, walk in shared_choices(plan, calls)]
