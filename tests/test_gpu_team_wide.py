"""The widest team launches, with vectors beside the registers in LDS, against the
streaming kernels: p(3)-CG with four unknowns per thread, 3D CG with six."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,method,l", [
    ((1000, 901), "plcg", 3), ((1024, 960), "plcg", 3), ((101, 97, 89), "plcg", 3),
    ((64, 120, 118), "plcg", 3), ((128, 101, 97), "cg", 1), ((127, 113, 99), "cg", 1)])
@pytest.mark.parametrize("maxit", [3, 80])
def test_iterates(dims, method, l, maxit):
    """The iterates of the streaming kernels to 1e-11 (rounding of sums of 10^6 terms, grown
    over at most 80 iterations); repeated solves the same bits."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_06850_amd import plcg
    print(f"[gpu] wide {method} l={l} dims={dims} maxit={maxit}", flush=True)
    n = int(np.prod(dims))
    b = torch.from_numpy(synth.uniform(n, 3)).to("cuda:0")
    out = []
    for launch in ("auto", "auto", "streaming"):
        s = plcg.Solver("2d5" if len(dims) == 2 else "3d7", dims, method=method, l=l, lmin=0.0,
                        lmax=8.0 if len(dims) == 2 else 12.0, launch=launch)
        x = torch.zeros_like(b)
        r = s.solve(b, x, 1e-30, maxit)
        s.close()
        out.append((x.cpu().numpy(), r))
    (x, r), (x2, _), (y, q) = out
    assert np.array_equal(x, x2)
    assert r.iters == q.iters == maxit and r.reason == q.reason
    assert np.linalg.norm(x - y) <= 1e-11 * np.linalg.norm(y)
    assert r.host_waits <= 5
