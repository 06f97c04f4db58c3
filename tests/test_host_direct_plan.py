"""Host logic: which tile of the direct kernel a call takes (csrc/direct_plan.h), on measured calls.  Compiled for the host
with g++ and run here; no GPU involved."""
import os
import subprocess

import pytest

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
