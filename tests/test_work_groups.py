"""The rule that sizes the page kernels' work items, at rounds on both sides of its lines (host code, no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_agents_per_work_item(tmp_path):
    exe = str(tmp_path / "work_group_check")
    csrc = os.path.join(ROOT, "paper_2604_03143_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", csrc,
           os.path.join(ROOT, "tests", "work_group_check.cpp"), os.path.join(csrc, "tdk_plan.cpp"), "-o", exe]
    subprocess.run(cmd, check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
