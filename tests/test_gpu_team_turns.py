"""Team launches of many solves and a batch at once, from a thread each: those that fit on the GPU
together run beside each other, none is lost to another, and each gives the bits it gives
alone."""
import threading

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

# one workgroup; two and twenty on one XCD; more than half and nearly all of the device
SOLVES = [((37, 53), "cg", 1), ((60, 40), "plcg", 2), ((64, 64), "plcg", 2), ((100, 80), "cg", 1),
          ((300, 200), "plcg", 1), ((513, 301), "cg", 1), ((60, 50, 40), "plcg", 3),
          ((1024, 1024), "plcg", 1)]


def test_solves_and_a_batch_at_once():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_06850_amd import plcg
    dev = torch.device("cuda:0")

    def solve(k, out, reps):
        dims, method, l = SOLVES[k]
        stream = torch.cuda.Stream(dev)
        with torch.cuda.stream(stream):
            s = plcg.Solver("2d5" if len(dims) == 2 else "3d7", dims, method=method, l=l,
                            lmax=8.0 if len(dims) == 2 else 12.0)
            b = torch.from_numpy(synth.uniform(int(np.prod(dims)), k)).to(dev)
            for _ in range(reps):
                x = torch.zeros_like(b)
                r = s.solve(b, x, 1e-8, 400, stream.cuda_stream)
                stream.synchronize()
                out.append((r.iters, r.host_waits, x))
            s.close()

    alone = []
    for k in range(len(SOLVES)):
        out = []
        solve(k, out, 1)
        alone.append(out[0])
        assert out[0][1] == 3                 # setup, the launch, the final residual
    dims = [(150, 140), (64, 90), (90, 33)]
    coef = [synth.edge_coefficients(d, 7 + k) for k, d in enumerate(dims)]
    bs = [torch.from_numpy(synth.uniform(d[0] * d[1], 20 + k)).to(dev) for k, d in enumerate(dims)]

    def batch(out):
        stream = torch.cuda.Stream(dev)
        with torch.cuda.stream(stream):
            q = plcg.Batch(l=2, max_slots=3, arena_bytes=1 << 28)
            xs = [torch.zeros_like(b) for b in bs]
            stream.synchronize()
            ts = [q.add(d, b.data_ptr(), x.data_ptr(), 1e-9, 5000, stream.cuda_stream, c[0], c[1])
                  for d, b, x, c in zip(dims, bs, xs, coef)]
            done = {}
            for _ in range(2000):
                q.step(16, stream.cuda_stream)
                stream.synchronize()
                for k, t in enumerate(ts):
                    if k not in done:
                        r = q.poll(t)
                        if r is not None:
                            done[k] = r.iters
                if len(done) == 3:
                    break
            q.close()
            out.append((done, xs))

    ref = []
    batch(ref)
    torch.cuda.synchronize()
    got = [[] for _ in SOLVES]
    runs = []
    print("[gpu] eight solvers and a batch at once", flush=True)
    threads = [threading.Thread(target=solve, args=(k, got[k], 6)) for k in range(len(SOLVES))]
    threads += [threading.Thread(target=batch, args=(runs,)) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    for k, out in enumerate(got):
        assert len(out) == 6
        for iters, waits, x in out:
            assert (iters, waits) == alone[k][:2], SOLVES[k]      # no launch was given up
            assert torch.equal(x, alone[k][2]), SOLVES[k]
    assert len(runs) == 2
    for done, xs in runs:
        assert done == ref[0][0]
        assert all(torch.equal(x, y) for x, y in zip(xs, ref[0][1]))
