"""The epsilon rule's run search on long axes whose prefix sums lose mass
(tests/host/eps_run_long.cpp), built with g++ (no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_run_search_on_long_axes(tmp_path):
    exe = str(tmp_path / "eps")
    cmd = ["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2208_06097_amd", "csrc"), os.path.join(HERE, "host", "eps_run_long.cpp"),
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout + r.stderr)
    assert r.returncode == 0 and "long axes: 0 failures" in r.stdout
