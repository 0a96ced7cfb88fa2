"""The workgroups of the pre-pass launches (no GPU needed)."""
import os
import subprocess

from paper_2603_02170_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_prepass_launches_take_every_block_once(tmp_path):
    exe = str(tmp_path / "prepass_order")
    cmd = [build.hipcc_path(), "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2603_02170_amd", "csrc"),
           os.path.join(ROOT, "tests", "prepass_order.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
