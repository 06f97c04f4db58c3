"""Host logic: how the kernels whose weights stay in LDS split a call and which calls take them (csrc/resident_plan.h), that their GPU
tests' calls do, and that the calls of the other kernels' tests on plain bits do not.  Compiled for the host with g++."""
import os
import subprocess

import pytest

import test_gpu_direct_tiles as T
import test_gpu_resident as R
import test_gpu_shared_weights as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("resident_plan") / "resident_plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_00704_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "resident_plan_check.cpp"), "-o", exe], check=True)
    return exe


def test_every_column_is_taken_once(checker):
    out = subprocess.run([checker], stdout=subprocess.PIPE, text=True, timeout=300)
    assert out.returncode == 0, out.stdout


def ask(checker, rows, what):
    out = subprocess.run([checker, what], input="\n".join(" ".join(str(int(v)) for v in r) for r in rows), stdout=subprocess.PIPE, text=True, check=True)
    return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]


def takes(checker, calls):
    """Per call (n, c_in, h, w, c_out, filter, stride, pad): whether the kernel takes it, words of a load."""
    return ask(checker, [(n * ((h + 2 * p - k) // st + 1) * ((w + 2 * p - k) // st + 1), o, (c + 31) // 32, k * k, 1, 0, 0) for n, c, h, w, o, k, st, p in calls],
               "calls")


def takes_branches(checker, calls, out, nothing_outside=False, own=R.own_tensors):
    """The same per call (n, c_in, h, w, c_out, taps, stride) of branches."""
    return ask(checker, [(n * ((h - 1) // st + 1) * ((w - 1) // st + 1), o, (c + 31) // 32, t, out == "bits", own(t), nothing_outside) for n, c, h, w, o, t, st in calls],
               "branches")


def test_calls_of_the_gpu_tests(checker):
    mine = [(n, c, h, w, o, 3, st, p) for _, (n, c, h, w, o, st, p) in R.CALLS]
    assert takes(checker, mine) == [(1, wide) for wide, _ in R.CALLS]
    others = [(n, c, h, w, o, k, 1, k // 2) for kind, _, _, (n, c, h, w, o, k) in T.CONVS if kind == T.BITS]
    others += [(n, c, h, w, o, k, st, k // 2) for kind, _, _, (n, c, h, w, o, k, st) in S.CONVS + S.ALIGNED if kind == S.BITS]
    assert not any(t for t, _ in takes(checker, others))


def test_measured_calls(checker):
    ahead = [(64, 256, 28, 28, 256, 3, 1, 1), (64, 256, 56, 56, 512, 3, 2, 1), (512, 256, 28, 28, 256, 3, 1, 1)]
    behind = [(1, 256, 54, 54, 17637, 3, 2, 1), (344, 194, 9, 9, 9404, 3, 1, 1), (28, 160, 48, 48, 18528, 3, 2, 1), (13, 256, 31, 31, 5650, 3, 1, 1),
              (8, 297, 19, 19, 1408, 3, 1, 1), (13, 256, 28, 28, 288, 3, 1, 1), (37, 320, 37, 37, 32, 3, 1, 1), (146, 384, 41, 41, 32, 3, 1, 1), (13, 320, 27, 27, 200, 3, 1, 1), (64, 512, 14, 14, 256, 1, 1, 0)]
    assert [t for t, _ in takes(checker, ahead + behind)] == [1] * len(ahead) + [0] * len(behind)


def test_branch_calls_of_the_gpu_tests(checker):
    calls = [shape for _, shape in R.BRANCHES]
    for out in R.OUTS:
        assert takes_branches(checker, calls, out) == [(int(out == "bits" or (shape[5] > 5 and not R.own_tensors(shape[5]))), wide) for wide, shape in R.BRANCHES]
        assert takes_branches(checker, [s for _, s in R.BRANCHES_OF_TWO_LOADS], out) == [(0, wide) for wide, _ in R.BRANCHES_OF_TWO_LOADS]
        assert not any(t for t, _ in takes_branches(checker, calls, out, nothing_outside=True))
    # last columns that end inside their first 16 pixels (one lane half) and inside the others
    ends = [n * ((h - 1) // st + 1) * ((w - 1) // st + 1) % 32 for (n, _, h, w, _, _, st), (t, _) in zip(calls, takes_branches(checker, calls, "f32")) if t]
    assert any(0 < e < 16 for e in ends) and any(e > 16 for e in ends)
    ahead = [(64, 256, 28, 28, 256, 9, 1), (40, 320, 27, 27, 200, 9, 1), (64, 256, 28, 28, 256, 3, 1)]
    assert [t for t, _ in takes_branches(checker, ahead, "bits")] == [1, 1, 1]
    assert [t for t, _ in takes_branches(checker, ahead, "f32")] == [1, 1, 0]
    own = [(492, 160, 24, 24, 192, 4, 1), (37, 192, 40, 40, 512, 9, 1), (64, 256, 28, 28, 256, 9, 1)]
    assert [t for t, _ in takes_branches(checker, own, "f32", own=lambda taps: True)] == [0, 0, 0]
    assert [t for t, _ in takes_branches(checker, own, "bits", own=lambda taps: True)] == [1, 1, 1]
    few_taps = [(487, 225, 14, 14, 256, 5, 1), (58, 161, 30, 30, 704, 4, 1)]
    assert not any(t for t, _ in takes_branches(checker, few_taps, "f32", own=lambda taps: False))
    whole_taps_a_wave = [(3, 256, 49, 49, 96, 9, 1), (3, 227, 49, 49, 73, 9, 1), (2, 256, 33, 33, 352, 9, 1), (5, 192, 31, 31, 132, 4, 1)]
    assert not any(t for out in R.OUTS for t, _ in takes_branches(checker, whole_taps_a_wave, out))
    many_channels = [(41, 192, 21, 21, 9172, 3, 1), (1, 192, 36, 36, 18275, 9, 1), (4, 218, 28, 28, 17775, 9, 1)]
    assert not any(t for out in R.OUTS for t, _ in takes_branches(checker, many_channels, out))
    small = [(1, 256, 28, 28, 256, 9, 1), (2, 384, 13, 13, 384, 9, 1), (64, 128, 28, 28, 256, 9, 1)]
    assert not any(t for t, _ in takes_branches(checker, small, "bits"))
