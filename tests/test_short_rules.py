"""The rules of the one-launch forms of short heads (no GPU needed)."""
import os
import subprocess

from paper_2603_02170_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_faster_form_is_taken(tmp_path):
    exe = str(tmp_path / "short_rules")
    cmd = [build.hipcc_path(), "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2603_02170_amd", "csrc"),
           os.path.join(ROOT, "tests", "short_rules.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
