"""Team launches of batched systems: the sweeps of FP64 systems with l = 2 or 3 run many
to a launch, their vectors in registers.  Compared with the ticks, which run the sweeps
within a stream capture, and with themselves cut into launches another way."""
import threading

import numpy as np
import pytest
import torch

import synth
from oracle import operators

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


def _system(dims, seed):
    cx, cy, cz = synth.edge_coefficients(dims, seed)
    n = int(np.prod(dims))
    return {"dims": dims, "cx": cx, "cy": cy, "cz": cz, "b": synth.uniform(n, seed + 1), "n": n}


class Run:
    """Systems in one batch; step() until all are done."""

    def __init__(self, dev, systems, l, tol=1e-9, maxit=20000, use_graph=False, stream=None):
        from paper_1905_06850_amd import plcg
        self.stream = torch.cuda.current_stream(dev) if stream is None else stream
        self.batch = plcg.Batch(l=l, max_slots=len(systems), arena_bytes=1 << 30,
                                use_graph=use_graph)
        self.bufs, self.open, self.done = [], {}, {}
        with torch.cuda.stream(self.stream):
            for k, s in enumerate(systems):
                b = torch.from_numpy(s["b"]).to(dev)
                x = torch.zeros(s["n"], dtype=torch.float64, device=dev)
                t = self.batch.add(s["dims"], b.data_ptr(), x.data_ptr(), tol, maxit,
                                   self.stream.cuda_stream, s["cx"], s["cy"], s["cz"])
                assert t is not None
                self.bufs.append((b, x))
                self.open[t] = k

    def step(self, ticks):
        self.batch.step(ticks, self.stream.cuda_stream)

    def poll(self):
        self.stream.synchronize()
        for t in list(self.open):
            r = self.batch.poll(t)
            if r is not None:
                self.done[self.open.pop(t)] = r
        return not self.open

    def finish(self, ticks=16):
        for _ in range(20000):
            self.step(ticks)
            if self.poll():
                break
        assert not self.open
        out = [(self.done[k], x.cpu().numpy()) for k, (_, x) in enumerate(self.bufs)]
        self.batch.close()
        return out


# one tile and one more than its 64 columns or 45 rows (3D: 64 x 5 x 9 and its like); a
# last tile of one row; odd and narrow grids; the smallest; several tiles each way
EDGES = [(64, 45), (65, 45), (64, 46), (130, 91), (63, 136), (33, 17), (6, 5), (17, 300),
         (64, 5, 9), (65, 6, 10), (20, 31, 7), (4, 3, 3), (70, 40, 33)]


@pytest.mark.parametrize("l", [2, 3])
def test_team_sweeps_equal_the_ticks(dev, l):
    """Every system by team launches, by ticks, and from one to the other and back: x to
    1e-8 (what two solves stopped one iteration apart may differ by), iterations to 1."""
    systems = [_system(d, 10 * k + 1) for k, d in enumerate(EDGES)]
    team = Run(dev, systems, l).finish()

    def captured(lead, replays):
        """`lead` steps of 2 ticks, then `replays` replays of 20 captured ticks."""
        run = Run(dev, systems, l, stream=torch.cuda.Stream(dev))
        for _ in range(lead):
            run.step(2)
        run.stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=run.stream):
            run.step(20)
        with torch.cuda.stream(run.stream):
            for _ in range(replays):
                g.replay()
        run.stream.synchronize()
        return run

    ticks = captured(1, 60)
    assert ticks.poll()
    for run in (ticks, captured(12, 2)):
        for k, (r, x) in enumerate(run.finish() if run.open else
                                   [(run.done[j], b[1].cpu().numpy())
                                    for j, b in enumerate(run.bufs)]):
            rt, xt = team[k]
            assert r.reason == rt.reason == 1, (EDGES[k], r.as_dict(), rt.as_dict())
            assert abs(r.iters - rt.iters) <= 1 and r.restarts == rt.restarts
            assert np.linalg.norm(x - xt) <= 1e-8 * np.linalg.norm(xt), EDGES[k]
    for k, s in enumerate(systems):     # and x solves the system
        A, _, _ = operators.variable_laplacian(s["dims"], s["cx"], s["cy"], s["cz"])
        rel = np.linalg.norm(s["b"] - A(team[k][1])) / np.linalg.norm(s["b"])
        assert abs(rel - team[k][0].true_relres) <= 1e-3 * rel + 1e-14


@pytest.mark.parametrize("l", [2, 3])
@pytest.mark.parametrize("maxit", [20000, 0, 1, 2, 3, 40, 64])
def test_where_a_launch_ends_changes_nothing(dev, l, maxit):
    """Launches of 1, 5 and 64 sweeps, graph replay among the ticks, solves cut short by
    maxit around a launch's end: the same bits."""
    dims = [(64, 45), (96, 96), (130, 91), (20, 31, 7), (70, 40, 33)]
    systems = [_system(d, 10 * k + 5) for k, d in enumerate(dims)]
    ref = Run(dev, systems, l, maxit=maxit).finish(16)
    for ticks, graph in ((1, False), (5, False), (40, True)):
        if ticks == 1 and maxit > 64:
            continue
        for k, (r, x) in enumerate(Run(dev, systems, l, maxit=maxit, use_graph=graph).finish(ticks)):
            assert r.as_dict() == ref[k][0].as_dict(), (ticks, dims[k])
            assert np.array_equal(x, ref[k][1]), (ticks, dims[k])


def test_systems_beyond_one_launch_and_beside_streaming_ones(dev):
    """60 systems of 2 to 12 tiles need several launches a step, and one of 901 x 901 (280
    tiles) none: each result is the one it has alone."""
    dims = [(66 + 3 * (k % 20), 50 + 7 * (k % 13)) for k in range(60)] + [(901, 901)]
    systems = [_system(d, 3 * k + 1) for k, d in enumerate(dims)]
    mix = Run(dev, systems, 2, maxit=150).finish()
    for k in (0, 17, 39, 59, 60):
        r, x = Run(dev, [systems[k]], 2, maxit=150).finish(7)[0]
        assert r.as_dict() == mix[k][0].as_dict() and np.array_equal(x, mix[k][1]), dims[k]


def test_batches_and_solves_on_other_streams(dev):
    """Two batches on streams of their own, and a solve by team launch in a thread beside
    them: each as alone."""
    from paper_1905_06850_amd import plcg
    sets = [[_system(d, 7 * k + j) for k, d in enumerate([(150, 140), (64, 90), (90, 33)])]
            for j in (1, 2)]
    alone = [Run(dev, s, 2).finish() for s in sets]
    b = torch.from_numpy(synth.uniform(200 * 150, 3)).to(dev)
    solver = plcg.Solver("2d5", (200, 150), l=2)
    xref = torch.zeros_like(b)
    solver.solve(b, xref, 1e-9, 5000)
    torch.cuda.synchronize()
    got = []

    def solve():
        stream = torch.cuda.Stream(dev)
        with torch.cuda.stream(stream):
            for _ in range(5):
                x = torch.zeros_like(b)
                solver.solve(b, x, 1e-9, 5000)
                stream.synchronize()
                got.append(x)

    th = threading.Thread(target=solve)
    runs = [Run(dev, s, 2, stream=torch.cuda.Stream(dev)) for s in sets]
    th.start()
    for _ in range(2000):
        for r in runs:
            r.step(16)
        if all([r.poll() for r in runs]):
            break
    th.join()
    assert len(got) == 5 and all(torch.equal(x, xref) for x in got)
    for r, ref in zip(runs, alone):
        for k, (_, x) in enumerate(r.bufs):
            assert r.done[k].iters == ref[k][0].iters
            assert np.array_equal(x.cpu().numpy(), ref[k][1])
        r.batch.close()
