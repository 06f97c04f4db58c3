"""Host logic: how the direct kernel's branch mode walks a tap's packed words (csrc/branch_walk.h).  The checker
(tests/host/branch_walk_check.cpp) walks 1 to 4096 words through the functions the kernel itself uses: every word once,
none outside its tap, the zero positions as many as the start value allows for.  Compiled for the host with g++ and
run here; no GPU involved."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_branch_walk_reads_every_word_once(tmp_path):
    exe = str(tmp_path / "branch_walk_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_00704_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "branch_walk_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    assert "mismatches: 0" in out.stdout
