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
    """Per call: tile and words per load (0: another kernel) and the other choice's tile and walk; of branches: form, tile, words per load."""
    lines = "\n".join(" ".join(str(int(v)) for v in c) for c in calls)
    out = subprocess.run([checker, mode], input=lines, stdout=subprocess.PIPE, text=True, timeout=300, check=True)
    return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]


def call(kind, n, c, h, w, o, k, stride, staged=0):
    m = n * ((h - 1) // stride + 1) * ((w - 1) // stride + 1)
    return (m, o, (c + 31) // 32, k, stride, kind if kind < 2 else 2 if staged else 3, kind, staged)


def test_every_tile_and_width_is_reached_on_the_gpu(checker):
    got = choices(checker, [call(kind, *shape) for kind, _, _, shape in G.CONVS] + [call(kind, *shape, staged=1) for kind, _, _, shape in G.ALIGNED])
    assert [g[:2] for g in got] == [(tile, wide) for _, tile, wide, _ in G.CONVS + G.ALIGNED]
    grid = [(m, o, cw, ks, stride, kind if kind < 2 else 3, kind, 0) for m in (196, 784, 3136, 12544, 50176, 200704) for o in (16, 64, 100, 256, 512)
            for cw in (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 16, 18, 32) for ks in (1, 3) for stride in (1, 2) for kind in (G.BITS, G.SUMS, G.HALF, G.FLOAT)]
    grid += [(m, o, cw, ks, stride, kind if kind < 2 else 2 if o % 128 == 0 else 3, kind, 1) for m, o, cw, ks, stride, _, kind, _ in grid if cw % 4 == 0]
    listed = {(kind, tile, wide) for kind, tile, wide, _ in G.CONVS + G.ALIGNED}
    reached = {(c[6], tile, wide) for c, (tile, wide, _, _) in zip(grid, choices(checker, grid)) if tile}
    assert reached <= listed, sorted(reached - listed)


def test_every_branch_form_is_reached_on_the_gpu(checker):
    """Per kind of output, each a kernel of its own: every form, tile and, on shared weights, width of loads."""
    def tail(out):
        return out.startswith("module"), out == "module_f16"

    def kernel(form, tile, wide, out):
        return form, tile, wide if form == G.SHARED else 0, out

    calls = [(n * h * w, o, (c + 31) // 32, taps, *tail(out)) for _, _, _, out, (n, c, h, w, o, taps) in G.BRANCHES]
    assert choices(checker, calls, "branches") == [(form, tile, wide) for form, tile, wide, _, _ in G.BRANCHES]
    grid = [(out, (m, o, cw, p, *tail(out))) for m in (49, 784, 12544, 50176, 200704) for o in (32, 100, 256, 512, 1000)
            for cw in (1, 2, 3, 4, 5, 8, 9, 16, 32) for p in (1, 2, 3, 8, 9, 16) for out in G.OUTS]
    got = choices(checker, [c for _, c in grid], "branches")
    reached, listed = {kernel(*g, out) for (out, _), g in zip(grid, got)}, {kernel(*row[:4]) for row in G.BRANCHES}
    assert reached <= listed, sorted(reached - listed)


@pytest.mark.parametrize("kind,shared,call", [
    # pixels, channels out, words, filter, stride, whether the staged kernel covers the call; times in us of the other kernels and of this form
    ("half", False, (122713, 88, 4, 3, 1, 0)),           # 20.8, 23.0
    ("half", False, (45800, 70, 4, 3, 2, 0)),           # 11.5, 13.0
    ("half", False, (163057, 61, 33, 3, 1, 0)),           # 70.4, 78.5
    ("half", False, (47579, 416, 33, 3, 2, 0)),           # 123, 166
    ("float", False, (54000, 96, 35, 3, 2, 0)),           # 45.2, 64.4
    ("sums", False, (10976, 800, 34, 3, 1, 0)),           # 48.7, 63.1
    ("half", False, (9016, 268, 18, 3, 2, 0)),           # 14.8, 16.9
    ("sums", False, (15680, 544, 21, 3, 2, 0)),           # 35.0, 41.7
    ("half", True, (42000, 339, 3, 3, 2, 0)),           # 40.7, 31.3
    ("half", True, (41067, 576, 8, 3, 1, 1)),           # 59.2, 44.1
    ("half", True, (83000, 96, 16, 3, 2, 1)),           # 41.0, 31.3
    ("float", True, (83655, 96, 24, 3, 1, 1)),           # 52.1, 38.7
    ("sums", True, (84672, 315, 8, 3, 1, 1)),           # 152, 34.8
    ("half", False, (50176, 256, 32, 3, 1, 1)),           # 63.0, 66.8
    ("half", False, (32585, 512, 36, 3, 2, 1)),           # 82.8, 130
    ("half", False, (47040, 256, 36, 3, 2, 1)),           # 68.3, 97.2
    ("bits", False, (16611, 896, 36, 1, 2, 1)),           # 11.5, 16.5
    ("bits", True, (56316, 192, 10, 3, 1, 0)),           # 27.9, 16.3
])
def test_measured_calls_go_to_the_faster_form(checker, kind, shared, call):
    m, o, cw, ks, stride, staged = call
    other, mine = {"bits": (0, G.BITS), "sums": (1, G.SUMS), "half": (3, G.HALF), "float": (3, G.FLOAT)}[kind]
    (tile, *_), = choices(checker, [(m, o, cw, ks, stride, other, mine, staged)])
    assert (tile != 0) == shared


@pytest.mark.parametrize("out,form,tile,call", [
    # pixels, channels out, words, branches; times in us of the choice and of what it was measured against
    ("bits", G.OWN, None, (242452, 96, 3, 1)),              # 13.5, shared weights 16.4
    ("bits", G.OWN, None, (156333, 68, 3, 1)),              # 9.6, shared weights 11.6
    ("module_f16", G.SHARED, G.S_1X1, (184730, 81, 1, 9)),  # 51.0, 2 x 1 blocks 60.6
    ("module_f16", G.SHARED, G.S_1X1, (139239, 85, 2, 6)),  # 33.4, 2 x 1 blocks 38.2
    ("module_f16", G.SHARED, G.S_1X1, (22194, 142, 8, 8)),  # 17.2, 2 x 1 blocks 20.0
    ("module_f32", G.SHARED, G.S_1X1, (286117, 416, 3, 3)), # 199, 2 x 1 blocks 258
    ("module_f32", G.SHARED, G.S_1X1, (34983, 890, 3, 3)),  # 111, 2 x 1 blocks 134
    ("bits", G.SHARED, G.S_2X1, (50176, 256, 8, 9)),        # 21.5, 1 x 1 blocks 24.7
])
def test_measured_branch_calls_go_to_the_faster_form(checker, out, form, tile, call):
    (got, blocks, _), = choices(checker, [(*call, out.startswith("module"), out == "module_f16")], "branches")
    assert got == form and (tile is None or blocks == tile)
