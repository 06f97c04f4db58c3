"""Host logic: AUTO's rules for launches that their output binds (csrc/auto_plan.h), on measured calls.  Compiled for the
host with g++ and run here; no GPU involved."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_measured_calls_go_where_they_are_faster(tmp_path):
    exe = str(tmp_path / "auto_plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_00704_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "auto_plan_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    assert "mismatches: 0" in out.stdout
