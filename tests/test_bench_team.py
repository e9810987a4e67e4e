"""bench.py's account of solves that run in one launch per run: which those are, from the
host's waits, and a roofline of the bytes that they move."""
from types import SimpleNamespace

import pytest

import bench


@pytest.mark.parametrize("iters,restarts,waits,jacobi,team", [
    (2900, 0, 3, False, True), (2900, 0, 48, False, False), (64, 0, 3, False, True),
    (64, 0, 4, False, False), (850, 0, 4, True, True), (850, 0, 16, True, False),
    (400, 2, 7, False, True), (400, 2, 14, False, False), (40, 0, 3, False, False)])
def test_which_solves_are_team_runs(iters, restarts, waits, jacobi, team):
    r = SimpleNamespace(iters=iters, restarts=restarts, host_waits=waits)
    assert bench.team_run(r, False, jacobi) == team
    assert not bench.team_run(r, True, jacobi)


def test_roofline_of_a_team_run():
    # 1024^2 p(1): 2900 iterations of 4.05 us in one launch that reads x and z_0 and writes x
    n, iters = 1024 * 1024, 2900
    hr = {"launch": "team", "launches_per_iter": 1 / iters, "us_per_iter": 4.05,
          "bytes_per_iter": 24 * n / iters, "working_set_bytes": 0, "cache_resident": True}
    r = bench.roofline("poisson1024", "2d5", ("plcg", 1), hr)
    assert r["kernel"] == "plcg_team_kernel" and r["bound"] == "latency"
    assert r["bytes_per_launch"] == pytest.approx(24 * n)
    assert r["kernel_us"] == pytest.approx(4.05 * iters)
    assert r["frac"] == pytest.approx(24 * n / (4.05e-6 * iters) / 8e12, rel=1e-6)
