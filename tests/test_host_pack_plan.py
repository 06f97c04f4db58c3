"""Host logic: which calls the ballot pack takes and how its workgroups cover them (csrc/pack_plan.h).  The checker
(tests/host/pack_plan_check.cpp) walks the workgroups through the functions that launcher and kernel use.  Compiled for
the host with g++ and run here; no GPU involved."""
import os
import subprocess

import pytest

import test_gpu_pack_staged as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pack_plan") / "pack_plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_00704_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "pack_plan_check.cpp"), "-o", exe], check=True)
    return exe


def test_ballot_plan_covers_every_row_and_channel_once(checker):
    out = subprocess.run([checker], stdout=subprocess.PIPE, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    assert "mismatches: 0" in out.stdout


def ask(checker, calls):
    """Per (element bytes, address, outer, channels, source channels, inner): vectors of a row in the kernel through LDS or 0, loads past the caches' lines."""
    out = subprocess.run([checker, "staged"], input="\n".join(" ".join(map(str, c)) for c in calls), stdout=subprocess.PIPE, text=True, check=True)
    return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]


def form(row):
    return "vectors" if row % 16 == 0 else "dwords" if row % 4 == 0 else "bytes"


def test_calls_of_the_gpu_tests_go_through_lds(checker):
    calls = [(size, P.offset(n), n, rep * c, c, inner) for size in (4, 2, 1) for n, c, inner, rep in P.SHAPES]
    got = ask(checker, calls)
    for (size, _, _, _, c, inner), (vectors, _) in zip(calls, got):
        assert bool(vectors) == (16 < size * inner <= 208 and c * inner * size % 4 == 0), (size, c, inner)
    reached = {(size, vectors, form(size * inner)) for (size, _, _, _, _, inner), (vectors, _) in zip(calls, got) if vectors}
    assert {v for s, v, _ in reached if s == 4} == {2, 3, 4, 5, 6, 7, 8, 10, 13}
    assert {v for s, v, _ in reached if s == 2} == {2, 3, 4, 5, 6, 7, 8} and {v for s, v, _ in reached if s == 1} == {2, 3, 4}
    assert {(s, f) for s, _, f in reached} == {(4, "vectors"), (4, "dwords"), (2, "vectors"), (2, "dwords"), (2, "bytes"), (1, "vectors"), (1, "dwords"), (1, "bytes")}


def test_loads_past_the_caches_of_the_gpu_tests(checker):
    sizes = [(P.element_size(dtype), c, inner) for dtype, c, inner in P.BEYOND_THE_CACHE]
    whole = [(size, 0, P.images(size, c, inner), c, c, inner) for size, c, inner in sizes]
    parts = [(size, 0, n // 2, c, c, inner) for size, _, n, c, _, inner in whole]
    assert all(v and s for v, s in ask(checker, whole)) and all(v and not s for v, s in ask(checker, parts))
    assert {(size, form(size * inner)) for size, _, inner in sizes} == {(4, "vectors"), (4, "dwords"), (2, "vectors"), (2, "dwords"), (2, "bytes"), (1, "vectors"), (1, "bytes")}
    assert [s for _, s in ask(checker, [(4, 0, 512, 256, 256, 49), (4, 0, 515, 252, 252, 49)])] == [1, 1]      # float rows beyond seven vectors, from 16 MB on
