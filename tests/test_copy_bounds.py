"""The staging copies of the backward with one KV block per workgroup and with four stay inside the caller's tensors, for every small
(N_q, N_kv) with and without the mask, those of the forward with four waves per 32 queries and of dQ with one Q block per workgroup take the
tiles they are for, and every workgroup of a launch has one (head, item) of its own: the kernels' own
index functions, run on the host (no GPU needed)."""
import os
import subprocess

from paper_2603_02170_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_copied_row_and_every_work_item_exists(tmp_path):
    exe = str(tmp_path / "copy_bounds")
    cmd = [build.hipcc_path(), "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2603_02170_amd", "csrc"),
           os.path.join(ROOT, "tests", "copy_bounds.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
