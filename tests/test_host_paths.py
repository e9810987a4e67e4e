"""The host side of the library on a device made of host functions (tests/c/fake_device.h):
paths that a GPU takes seldom, such as launches that are given up, a full device, calls
under stream capture and several threads."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1905_06850_amd", "csrc")
ROCM = "/opt/rocm/include"


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(ROCM):
        pytest.skip("no host compiler or no HIP headers")
    d = tmp_path_factory.mktemp("host_paths")
    out = d / "host_paths"
    sources = [os.path.join(CSRC, f) for f in ("plcg_engine.cpp", "plcg_batch.cpp",
                                               "plcg_serve.cpp")]
    sources.append(os.path.join(ROOT, "tests", "c", "host_paths.cpp"))
    procs = [subprocess.Popen(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", ROCM,
                               "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", s,
                               "-o", str(d / f"{k}.o")]) for k, s in enumerate(sources)]
    assert all(p.wait() == 0 for p in procs)
    subprocess.run(["g++", "-pthread", *[str(d / f"{k}.o") for k in range(len(sources))],
                    "-o", str(out)], check=True)
    return str(out)


@pytest.mark.parametrize("scenario", ["lost_record", "step_counts", "step_counts_lost", "turns", "capture", "autotune",
                                      "no_mail", "few_ticks", "few_ticks_mixed", "rows_order", "x_updates", "which_team",
                                      "any_stencil", "no_iterations", "resident_3d",
                                      "thin_3d"])
def test_host_path(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
