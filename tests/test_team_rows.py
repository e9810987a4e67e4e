"""The cut of an assembled matrix's rows over a team launch (plcg_team.h), on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_row_has_one_place(tmp_path):
    exe = tmp_path / "team_rows"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_1905_06850_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "team_rows.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
