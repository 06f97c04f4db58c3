"""Host logic: which calls the ballot pack takes and how its workgroups cover them (csrc/pack_plan.h).  The checker
(tests/host/pack_plan_check.cpp) walks the workgroups through the functions that launcher and kernel use.  Compiled for
the host with g++ and run here; no GPU involved."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_ballot_plan_covers_every_row_and_channel_once(tmp_path):
    exe = str(tmp_path / "pack_plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_00704_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "pack_plan_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    assert "mismatches: 0" in out.stdout
