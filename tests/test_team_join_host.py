"""The formation of CG teams on the CPU: threads in the place of workgroups,
more of them than may run at a time, under the undefined-behaviour sanitizer
(tests/host/team_join.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_teams_are_whole_or_not_there(tmp_path):
    exe = str(tmp_path / "join")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "paper_2208_06097_amd", "csrc"), os.path.join(HERE, "host", "team_join.cpp"),
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(r.stdout + r.stderr)
    assert r.returncode == 0 and "team formation: 0 failures" in r.stdout
