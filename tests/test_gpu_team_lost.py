"""Team launches that do not get all their workgroups onto the GPU: a wave of other work
holds a compute unit that a launch of 256 tiles needs, longer than the launch waits.  The
launch ends by its bounded waits and the other kernels make the run."""
import time

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


class Holder:
    """One wave that occupies a compute unit for a time, on a stream of its own."""

    def __init__(self, dev):
        self.stream = torch.cuda.Stream(dev)
        self._sleep(1000)
        cycles = 2_000_000
        t0 = time.perf_counter()
        self._sleep(cycles)
        self.per_second = cycles / (time.perf_counter() - t0)

    def _sleep(self, cycles):
        with torch.cuda.stream(self.stream):
            torch.cuda._sleep(int(cycles))
        self.stream.synchronize()

    def hold(self, seconds):
        with torch.cuda.stream(self.stream):
            torch.cuda._sleep(int(seconds * self.per_second))
        time.sleep(0.05)       # it runs by now

    def wait(self):
        self.stream.synchronize()


@pytest.fixture(scope="module")
def holder(dev):
    return Holder(dev)


# plans of 256 tiles whose sixteen waves take all registers of a compute unit
@pytest.mark.parametrize("dims,method,l", [
    ((1024, 2300), "cg", 1), ((128, 60, 190), "cg", 1), ((128, 40, 230), "plcg", 1),
    ((1024, 901), "plcg", 2), ((1024, 901), "plcg", 3)])
@pytest.mark.parametrize("check_every", [0, 1])
def test_lost_solve_streams(dev, holder, dims, method, l, check_every):
    """x and the counts are, bit for bit, those of the streaming kernels, which make the run;
    so are those of the handle's next solve."""
    from paper_1905_06850_amd import plcg
    n = int(np.prod(dims))
    b = torch.from_numpy(synth.uniform(n, 5)).to(dev)
    kw = dict(method=method, l=l, lmax=8.0 if len(dims) == 2 else 12.0, check_every=check_every)
    kind = "2d5" if len(dims) == 2 else "3d7"
    print(f"[gpu] lost team launch {method} l={l} {dims} check_every={check_every}", flush=True)
    s = plcg.Solver(kind, dims, launch="streaming", **kw)
    ref = torch.zeros_like(b)
    rr = s.solve(b, ref, 1e-30, 100)
    s.close()
    s = plcg.Solver(kind, dims, **kw)
    for k in range(2):
        x = torch.zeros_like(b)
        torch.cuda.synchronize()
        if k == 0:
            holder.hold(0.5)
        r = s.solve(b, x, 1e-30, 100)
        holder.wait()
        assert (r.seconds > 0.2) == (k == 0)      # the first solve's launch waited, and gave up
        assert r.iters == rr.iters == 100 and r.reason == rr.reason
        assert r.rec_relres == rr.rec_relres and r.true_relres == rr.true_relres
        assert torch.equal(x, ref)
    s.close()


class _Batch:
    """Systems in a batch of their own, stepped until they are done."""

    def __init__(self, dev, dims, l, maxit, tol=1e-30, seed=3):
        from paper_1905_06850_amd import plcg
        self.stream = torch.cuda.current_stream(dev).cuda_stream
        self.batch = plcg.Batch(l=l, max_slots=len(dims), arena_bytes=1 << 30)
        self.x, self.b, self.tickets = [], [], []
        for k, d in enumerate(dims):
            n = int(np.prod(d))
            cx, cy, cz = synth.edge_coefficients(d, seed + k)
            self.b.append(torch.from_numpy(synth.uniform(n, seed + 50 + k)).to(dev))
            self.x.append(torch.zeros_like(self.b[-1]))
            self.tickets.append(self.batch.add(d, self.b[-1].data_ptr(), self.x[-1].data_ptr(),
                                               tol, maxit, self.stream, cx, cy, cz))
        torch.cuda.synchronize()

    def step(self, ticks=16):
        self.batch.step(ticks, self.stream)

    def finish(self):
        done, steps = {}, 0
        while len(done) < len(self.tickets):
            self.step()
            torch.cuda.synchronize()
            steps += 1
            assert steps < 2000
            for k, t in enumerate(self.tickets):
                if k not in done:
                    r = self.batch.poll(t)
                    if r is not None:
                        done[k] = r
        self.batch.close()
        return [done[k] for k in range(len(done))], [x.cpu().numpy() for x in self.x], steps


# one system of 256 tiles whose waves take all registers, alone and beside a small one
@pytest.mark.parametrize("dims,l", [([(1024, 720)], 3), ([(64, 80, 140), (30, 20, 10)], 2)])
@pytest.mark.parametrize("lead", [1, 3])
def test_lost_batch_goes_on(dev, holder, dims, l, lead):
    """A launch lost after `lead` steps: no x-update is lost or made twice, x is that of a
    batch whose launches all ran (to 1e-8, as the ticks' x in test_gpu_team_batch.py)."""
    print(f"[gpu] lost batch launch {dims} l={l} after {lead} steps", flush=True)
    ref, xref, _ = _Batch(dev, dims, l, 300).finish()
    run = _Batch(dev, dims, l, 300)
    for _ in range(lead):
        run.step()
    torch.cuda.synchronize()
    holder.hold(0.6)
    t0 = time.perf_counter()
    run.step()
    torch.cuda.current_stream(dev).synchronize()
    assert time.perf_counter() - t0 > 0.2
    holder.wait()
    got, x, steps = run.finish()
    # 16 x-updates a step are left to the ticks, beside setup, fill and report
    assert steps <= (300 + 10 + l) // 16 + 2
    for k in range(len(dims)):
        assert got[k].iters == ref[k].iters and got[k].restarts == ref[k].restarts
        assert got[k].reason == ref[k].reason
        assert np.linalg.norm(x[k] - xref[k]) <= 1e-8 * np.linalg.norm(xref[k])
