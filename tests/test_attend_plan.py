"""The attention planner (which kernels, how the span is cut, launch sizes, workspace layout) is host code without HIP: a
native driver checks it over random shapes under AddressSanitizer and UBSan."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan"]


def test_attention_planner_under_asan_and_ubsan(tmp_path):
    exe = str(tmp_path / "attend_plan_check")
    csrc = os.path.join(ROOT, "paper_2604_03143_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-g", *SAN, "-I", os.path.join(ROOT, "include"), "-I", csrc,
           os.path.join(ROOT, "tests", "attend_plan_check.cpp"), os.path.join(csrc, "tdk_plan.cpp"), "-o", exe]
    subprocess.run(cmd, check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "clean" in run.stdout
