"""Team launches (a whole run in one launch of one workgroup per tile, what AUTO takes
for mid-size stencils) against the oracle, at the edges of the tiles: a lane more or
less than 64 columns, a row more or less than a tile, the last tile partly and whole
waves outside the grid, one tile and the most tiles, every width of unknowns per
thread."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from oracle import cg as ocg
from oracle import operators, shifts
from oracle import plcg as oplcg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _solve(dev, dims, method, l, b, tol, maxit, coef=None, launch="auto", repeat=1):
    from paper_1905_06850_amd import plcg
    print(f"[gpu] team {method} l={l} dims={dims} tol={tol} maxit={maxit} "
          f"{'var' if coef else 'const'} {launch}", flush=True)
    kw = dict(lmax=8.0 if len(dims) == 2 else 12.0)
    keep = []
    if coef is not None:
        keep = [None if c is None else torch.from_numpy(c).to(dev) for c in coef]
        kw = dict(lmax=2.0, jacobi=True,
                  coef=tuple(None if c is None else c.data_ptr() for c in keep))
    s = plcg.Solver("2d5" if len(dims) == 2 else "3d7", dims, method=method, l=l, lmin=0.0,
                    launch=launch, **kw)
    bt = torch.from_numpy(b).to(dev)
    xs, r = [], None
    for _ in range(repeat):
        xt = torch.zeros(b.size, dtype=torch.float64, device=dev)
        r = s.solve(bt, xt, tol, maxit)
        xs.append(xt.cpu().numpy())
    s.close()
    assert all(np.array_equal(x, xs[0]) for x in xs)
    return xs[0], r


def _oracle(dims, method, l, b, tol, maxit, coef=None):
    if coef is None:
        A, dis, hi = operators.laplacian(dims), 1.0, 8.0 if len(dims) == 2 else 12.0
    else:
        _, A, dis = operators.variable_laplacian(dims, *coef)
        hi = 2.0
    x0 = np.zeros(A.n)
    ref = (ocg.cg(A, dis * b, x0, tol, maxit) if method == "cg" else
           oplcg.plcg(A, dis * b, x0, l, shifts.chebyshev_shifts(l, 0.0, hi), tol, maxit))
    return dis * ref.x, ref


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


METHODS = [("cg", 1), ("plcg", 1), ("plcg", 2), ("plcg", 3)]
# 2D: one lane over and under a tile's 64 columns, rows around the tiles of every
# width, long and narrow grids; 3D: the same along each axis, y sides with and without mail
DIMS = [(63, 61), (64, 75), (64, 76), (65, 45), (65, 61), (129, 91), (127, 46), (40, 300),
        (700, 20), (33, 17, 9), (64, 16, 31), (65, 9, 14), (20, 64, 5), (130, 7, 13)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("method,l", METHODS)
@pytest.mark.parametrize("var", [False, True])
def test_team_early_iterates(dev, dims, method, l, var):
    """x after m steps to rounding (1e-13, as the streamed iterates: 20 steps of operators
    and recurrences of condition near one)."""
    coef = synth.edge_coefficients(dims, 11) if var else None
    b = synth.uniform(int(np.prod(dims)), 12)
    for m in (1, 2, 5, 20):
        x, r = _solve(dev, dims, method, l, b, 1e-30, m, coef)
        xr, ref = _oracle(dims, method, l, b, 1e-30, m, coef)
        assert r.iters == m == ref.iters and r.reason == 2
        assert _rel(x, xr) < 1e-13, (m, _rel(x, xr))


# every number of unknowns per thread and one of the largest systems of each method
@pytest.mark.parametrize("dims,method,l", [
    ((64, 100), "cg", 1), ((640, 640), "cg", 1), ((1100, 1000), "cg", 1), ((1500, 1367), "cg", 1),
    ((300, 210), "plcg", 1), ((1024, 1024), "plcg", 1), ((1200, 1100), "plcg", 1),
    ((200, 150), "plcg", 2), ((512, 500), "plcg", 2), ((1024, 1020), "plcg", 2),
    ((256, 255), "plcg", 3), ((760, 740), "plcg", 3), ((60, 50, 40), "plcg", 3),
    ((70, 80, 90), "plcg", 1), ((70, 80, 90), "plcg", 2), ((101, 97, 89), "cg", 1)])
def test_team_equals_streaming(dev, dims, method, l):
    """300 steps against the streaming kernels (the oracle is slow at these sizes): x to
    1e-11, ten times what scaling b by three moves it; three solves in a row give the
    same bits (mail of earlier runs is not read again)."""
    b = synth.uniform(int(np.prod(dims)), 13)
    x, r = _solve(dev, dims, method, l, b, 1e-30, 300, repeat=3)
    xs, rs = _solve(dev, dims, method, l, b, 1e-30, 300, launch="streaming")
    assert r.iters == rs.iters == 300
    assert r.host_waits < rs.host_waits          # one launch, not one per iteration
    assert _rel(x, xs) < 1e-11
    assert r.rec_relres == pytest.approx(rs.rec_relres, rel=1e-6)


@pytest.mark.parametrize("method,l", METHODS)
def test_team_stops_as_the_oracle(dev, method, l):
    """Convergence, a breakdown with restarts (interval far too wide) and a zero and a
    non-finite right-hand side through the team path."""
    from paper_1905_06850_amd import plcg
    dims = (100, 60)
    b = synth.uniform(6000, 14)
    x, r = _solve(dev, dims, method, l, b, 1e-9, 5000)
    xr, ref = _oracle(dims, method, l, b, 1e-9, 5000)
    assert r.reason == 1 and abs(r.iters - ref.iters) <= 1 and _rel(x, xr) < 1e-8
    x, r = _solve(dev, dims, method, l, np.zeros(6000), 1e-9, 10)
    assert r.iters == 0 and r.reason == 1 and not x.any()
    b2 = b.copy()
    b2[17] = np.nan
    with pytest.raises(plcg.PlcgError) as ei:
        _solve(dev, dims, method, l, b2, 1e-9, 10)
    assert ei.value.status == plcg.PLCG_E_NONFINITE
    if method == "plcg":
        s = plcg.Solver("2d5", dims, method="plcg", l=l, lmin=0.0, lmax=16.0)
        bt = torch.from_numpy(b).to(dev)
        xt = torch.zeros(6000, dtype=torch.float64, device=dev)
        r = s.solve(bt, xt, 1e-8, 20000)
        s.close()
        assert r.reason == 1 and r.true_relres < 1e-7


def test_team_solves_from_two_threads(dev):
    """Two handles solving at once from two threads (each launch needs the whole GPU: the
    library runs them one after the other) give the bits they give alone."""
    import threading
    from paper_1905_06850_amd import plcg
    dims, n = (300, 200), 60000
    alone, got = {}, {}
    for seed in (1, 2):
        alone[seed], _ = _solve(dev, dims, "plcg", 2, synth.uniform(n, seed), 1e-8, 5000)

    def work(seed):
        stream = torch.cuda.Stream(dev)
        with torch.cuda.stream(stream):
            s = plcg.Solver("2d5", dims, method="plcg", l=2)
            bt = torch.from_numpy(synth.uniform(n, seed)).to(dev)
            out = []
            for _ in range(5):
                xt = torch.zeros(n, dtype=torch.float64, device=dev)
                s.solve(bt, xt, 1e-8, 5000, stream.cuda_stream)
                out.append(xt.cpu().numpy())
            s.close()
            got[seed] = out

    threads = [threading.Thread(target=work, args=(seed,)) for seed in (1, 2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    for seed in (1, 2):
        assert all(np.array_equal(x, alone[seed]) for x in got[seed])
