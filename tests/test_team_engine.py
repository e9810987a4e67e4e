"""The team kernels' scalar step (engine_gather, engine_step), compiled for the
host and fed the dot products the oracle's p(l)-CG forms, against engine_column,
the general form: state and coefficients bit for bit."""
import os
import subprocess

import pytest

from test_engine_replay import HIPCC, ROOT, _cases, _record


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_team_step_equals_the_general_form(tmp_path):
    exe = str(tmp_path / "team_engine")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17",
                    "-ffp-contract=off", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1905_06850_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "team_engine.hip"), "-o", exe],
                   check=True, capture_output=True)
    cases = [c for c in _cases() if c[1] <= 3]
    lines = [str(len(cases))]
    for name, l, A, b, lo, hi in cases:
        sig, beta, abs_tol, cols, _ = _record(A, b, l, lo, hi, 1e-10)
        lines.append(f"{name} {l} {len(cols)} {beta!r} {abs_tol!r} " + " ".join(map(repr, sig)))
        lines += [f"{c} " + " ".join(repr(r) for r in raw) for c, raw in cols]
    inp = tmp_path / "raw.txt"
    inp.write_text("\n".join(lines) + "\n")
    proc = subprocess.run([exe, str(inp)], capture_output=True, text=True)
    assert proc.returncode == 0, proc.stdout + proc.stderr
    assert proc.stdout.count("identical") == len(cases)
