"""The rules that choose between forms of a kernel, run on the host (no GPU needed)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rules_take_the_faster_side_and_return_what_can_be_launched(tmp_path):
    exe = str(tmp_path / "dispatch_rules")
    cmd = [os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2603_02170_amd", "csrc"),
           os.path.join(ROOT, "tests", "dispatch_rules.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
