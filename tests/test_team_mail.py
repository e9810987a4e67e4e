"""The team kernels' cut of a grid into tiles and the addressing of their mail
(plcg_team.h), checked on the host: coverage, bounds, one writer and the right
reader per word."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_word_has_one_writer_and_the_right_reader(tmp_path):
    exe = tmp_path / "team_mail"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_1905_06850_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "team_mail.cpp"), "-o", str(exe)], check=True)
    cases = [(1, 2, 0, 200, 150, 1, 256), (0, 1, 0, 513, 301, 1, 256), (1, 1, 0, 1024, 1024, 1, 256),
             (1, 1, 0, 1025, 1024, 1, 256), (1, 3, 1, 60, 50, 40, 256), (0, 1, 1, 101, 97, 89, 256),
             (1, 2, 1, 64, 64, 64, 256), (1, 1, 1, 1, 1, 6000, 256), (1, 2, 1, 5000, 1, 1, 256),
             (1, 2, 0, 1, 5000, 1, 256), (0, 1, 0, 64, 76, 1, 256), (1, 1, 0, 65, 76, 1, 8),
             (0, 1, 1, 65, 2, 300, 256), (1, 4, 0, 200, 150, 1, 256), (1, 1, 0, 2048, 2048, 1, 256)]
    rng = random.Random(4)
    for _ in range(60):
        d3 = rng.randint(0, 1)
        dims = [rng.randint(1, 120 if d3 else 700) for _ in range(3)]
        cases.append((rng.randint(0, 1), rng.randint(1, 3), d3, *dims[:2], dims[2] if d3 else 1,
                      rng.choice([256, 256, 64, 32])))
    cases = [c[:3] + (k % 2 if k > 14 else 0,) + c[3:] for k, c in enumerate(cases)]
    text = "\n".join(" ".join(map(str, c)) for c in cases)
    r = subprocess.run([str(exe)], input=text, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-300:]
    plans = r.stdout.split("\n")[:len(cases)]
    # a pipeline too deep and a system too large have no plan
    assert all(p != "none" for p in plans[:3] + plans[4:7])
    assert plans[13] == "none" and plans[14] == "none"
