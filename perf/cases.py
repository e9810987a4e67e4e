"""Timed cases of the solver: what programs that link the library have it do.

Every case is a whole solve (or a burst of served solves) through the public
binding: right-hand side in, solution out, x0 = 0, stopped by the tolerance or by
an iteration budget.  The listed cases and `draw` cover the same ranges: 2D and 3D
constant stencils from a few hundred unknowns to 2048^2 and 256^3, with even, odd and
elongated grids; CG and p(l)-CG; FP64 and FP32-stored refinement;
variable-coefficient stencils, assembled CSR matrices, and bursts of requests to
the batched server.
"""
import math

import numpy as np
import torch

from paper_1905_06850_amd import plcg

# Above these sizes a drawn solve is given an iteration budget (an inexact inner
# solve of an outer iteration), as converging would take longer than the largest
# listed case does.
BUDGET_2D, BUDGET_3D, BUDGET_VAR = 1_000_000, 4_000_000, 300_000


def listed():
    return [
        # the README's small grid: one solve of a few hundred microseconds, many of
        # which follow each other in a parameter study
        dict(name="2d_64_p2", op="2d", nx=64, ny=64, nz=1, method="plcg", l=2, tol=1e-8,
             maxit=100000, prec="fp64"),
        # the smallest kind of call: a ragged patch solved by classic CG
        dict(name="2d_37x53_cg", op="2d", nx=37, ny=53, nz=1, method="cg", l=1, tol=1e-8,
             maxit=100000, prec="fp64"),
        # a plane problem inside a time loop: latency-bound
        dict(name="2d_200x150_p2", op="2d", nx=200, ny=150, nz=1, method="plcg", l=2, tol=1e-8,
             maxit=100000, prec="fp64"),
        # an odd grid of ordinary size with classic CG
        dict(name="2d_513x301_cg", op="2d", nx=513, ny=301, nz=1, method="cg", l=1, tol=1e-8,
             maxit=100000, prec="fp64"),
        # the 1024^2 point of the size sweep
        dict(name="2d_1024_p1", op="2d", nx=1024, ny=1024, nz=1, method="plcg", l=1, tol=1e-8,
             maxit=100000, prec="fp64"),
        # the headline problem: 4 million unknowns, p(1)-CG
        dict(name="2d_2048_p1", op="2d", nx=2048, ny=2048, nz=1, method="plcg", l=1, tol=1e-8,
             maxit=100000, prec="fp64"),
        # a small box with a deeper pipeline
        dict(name="3d_60x50x40_p3", op="3d", nx=60, ny=50, nz=40, method="plcg", l=3, tol=1e-8,
             maxit=100000, prec="fp64"),
        # an ordinary box with odd sides
        dict(name="3d_101x97x89_cg", op="3d", nx=101, ny=97, nz=89, method="cg", l=1, tol=1e-8,
             maxit=100000, prec="fp64"),
        # the 256^3 problem in its fastest form: FP32 storage in FP64 refinement
        dict(name="3d_256_p1_fp32", op="3d", nx=256, ny=256, nz=256, method="plcg", l=1,
             tol=1e-10, maxit=100000, prec="fp32"),
        # a heterogeneous medium: lognormal edge coefficients, Jacobi-preconditioned
        dict(name="var2d_400x300_p2", op="var2d", nx=400, ny=300, nz=1, method="plcg", l=2,
             tol=1e-8, maxit=100000, prec="fp64"),
        # the same kind of operator handed over as an assembled matrix
        dict(name="csr_300x201_p1", op="csr", nx=300, ny=201, nz=1, method="plcg", l=1, tol=1e-8,
             maxit=100000, prec="fp64"),
        # a burst of requests on registered operators, sides 32..256
        dict(name="serve_24", op="serve", count=24, lo=32, hi=256, l=2, tol=1e-8, maxit=100000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["2d"] * 4 + ["3d"] * 3 + ["var2d"] * 2 + ["csr", "serve"])
    if kind == "serve":
        hi = rng.randint(96, 256)
        return dict(op="serve", count=rng.randint(6, 24), lo=rng.randint(24, 64), hi=hi,
                    l=rng.choice([2, 2, 3]), tol=1e-8, maxit=100000)
    method, l = rng.choice([("cg", 1), ("plcg", 1), ("plcg", 2), ("plcg", 2), ("plcg", 3)])
    prec = "fp64"
    nz = 1
    if kind == "3d":
        nx, ny, nz = (_log_int(rng, 10, 256) for _ in range(3))
        budget, mean = BUDGET_3D, 300
    elif kind == "2d":
        nx, ny = _log_int(rng, 24, 2048), _log_int(rng, 24, 2048)
        budget, mean = BUDGET_2D, 800
    elif kind == "var2d":
        nx, ny = _log_int(rng, 32, 1024), _log_int(rng, 32, 1024)
        budget, mean = BUDGET_VAR, 800
    else:
        nx, ny = _log_int(rng, 32, 512), _log_int(rng, 32, 512)
        budget, mean = BUDGET_VAR, 800
    if kind == "3d" and method == "plcg" and nx * ny * nz > 200_000 and rng.random() < 0.25:
        prec = "fp32"
    big = nx * ny * nz > budget
    return dict(op=kind, nx=nx, ny=ny, nz=nz, method=method, l=l,
                tol=1e-10 if prec == "fp32" else 1e-8,
                maxit=rng.randint(mean // 2, mean) if big and prec == "fp64" else 100000,
                prec=prec)


def _dims(case):
    return (case["nx"], case["ny"], case["nz"]) if case["op"] == "3d" else (case["nx"], case["ny"])


def _device():
    return torch.device("cuda:0")


def _rhs(n, seed):
    g = torch.Generator(device=_device())
    g.manual_seed(2 * seed + 1)
    return 2.0 * torch.rand(n, dtype=torch.float64, device=_device(), generator=g) - 1.0


def _edges(nx, ny, seed):
    """Lognormal(0, 1) edge coefficients cx (ny, nx+1) and cy (ny+1, nx)."""
    g = torch.Generator(device=_device())
    g.manual_seed(2 * seed + 2)
    cx = torch.randn(ny, nx + 1, dtype=torch.float64, device=_device(), generator=g).exp()
    cy = torch.randn(ny + 1, nx, dtype=torch.float64, device=_device(), generator=g).exp()
    return cx, cy


def _diagonal(cx, cy):
    return cx[:, :-1] + cx[:, 1:] + cy[:-1] + cy[1:]


def _assemble(cx, cy):
    """CSR arrays of the 5-point operator of edge coefficients cx, cy."""
    ny, nx = cy.shape[0] - 1, cy.shape[1]
    idx = torch.arange(nx * ny, device=cx.device).reshape(ny, nx)
    rows, cols, vals = [idx], [idx], [_diagonal(cx, cy)]
    for a, b, c in ((idx[:, :-1], idx[:, 1:], cx[:, 1:-1]), (idx[:-1], idx[1:], cy[1:-1])):
        rows += [a, b]
        cols += [b, a]
        vals += [-c, -c]
    rows, cols, vals = (torch.cat([t.reshape(-1) for t in v]) for v in (rows, cols, vals))
    order = torch.argsort(rows * (nx * ny) + cols)
    rowptr = torch.zeros(nx * ny + 1, dtype=torch.int64, device=cx.device)
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=nx * ny), 0)
    return rowptr, cols[order].to(torch.int32), vals[order].contiguous()


def _sides(case, seed=0):
    """Grid sizes of a burst: part of the case, not of the seed."""
    r = np.random.RandomState(7 * case["count"] + case["lo"] + case["hi"])
    return [(int(a), int(b)) for a, b in r.randint(case["lo"], case["hi"] + 1, (case["count"], 2))]


class State:
    pass


def prepare(case, seed):
    s = State()
    s.case = case
    if case["op"] == "serve":
        sides = _sides(case)
        l = case["l"]
        room = sum((2 * l + 4) * (nx * ny * 8 + 131072) for nx, ny in sides)
        s.batch = plcg.Batch(l=l, max_slots=len(sides), arena_bytes=2 * room, use_graph=True)
        s.ops, s.b, s.x = [], [], []
        for k, (nx, ny) in enumerate(sides):
            cx, cy = (c.cpu().numpy().reshape(-1) for c in _edges(nx, ny, seed * 1000 + k))
            s.ops.append(s.batch.register((nx, ny), cx, cy))
            s.b.append(_rhs(nx * ny, seed * 1000 + k))
            s.x.append(torch.empty(nx * ny, dtype=torch.float64, device=_device()))
        s.requests = [(0.0, k, case["maxit"], case["tol"], x.data_ptr()) for k, x in enumerate(s.x)]
        s.stream = torch.cuda.current_stream().cuda_stream
        torch.cuda.synchronize()
        return s
    dims = _dims(case)
    n = math.prod(dims)
    kw = dict(method=case["method"], l=case["l"], lmin=0.0, precision=case["prec"],
              inner_tol=1e-4 if case["prec"] == "fp32" else 0.0)
    s.b = _rhs(n, seed)
    s.x = torch.empty_like(s.b)
    if case["op"] == "2d":
        s.solver = plcg.Solver("2d5", dims, lmax=8.0, **kw)
    elif case["op"] == "3d":
        s.solver = plcg.Solver("3d7", dims, lmax=12.0, **kw)
    else:
        cx, cy = _edges(*dims, seed)
        if case["op"] == "var2d":
            torch.cuda.synchronize()
            s.solver = plcg.Solver("2d5", dims, lmax=2.0, jacobi=True,
                                   coef=(cx.data_ptr(), cy.data_ptr(), None), **kw)
        else:
            rowptr, colind, vals = _assemble(cx, cy)
            torch.cuda.synchronize()
            s.solver = plcg.Solver("csr", (n,), lmax=2.0, jacobi=True,
                                   csr=(rowptr.data_ptr(), colind.data_ptr(), vals.data_ptr(),
                                        vals.numel()), **kw)
    return s


def run(s):
    case = s.case
    if case["op"] == "serve":
        s.batch.serve(s.ops, [b.data_ptr() for b in s.b], s.requests, 16, 60.0, s.stream)
        return s.x
    s.x.zero_()
    s.solver.solve(s.b, s.x, case["tol"], case["maxit"])
    return s.x


def _iterations(case, dims):
    """About how many CG iterations the solve takes."""
    side = 1.0 / math.sqrt(sum(1.0 / (d + 1) ** 2 for d in dims) / len(dims))
    spread = 1.4 if case["op"] in ("var2d", "csr", "serve") else 1.0
    return min(case["maxit"], 0.25 * spread * (2 * side / math.pi) * math.log(2 / case["tol"]))


def work(case):
    """b read and x written once with the operator's data; CG's operations per iteration
    (operator, two products, three vector updates)."""
    if case["op"] == "serve":
        total = {"bytes": 0.0, "flops": 0.0}
        for dims in _sides(case):
            n = math.prod(dims)
            total["bytes"] += 8.0 * n * 4
            total["flops"] += 20.0 * n * _iterations(case, dims)
        return total
    dims = _dims(case)
    n = math.prod(dims)
    data = {"var2d": 16.0, "csr": 60.0}.get(case["op"], 0.0)
    apply = {"2d": 6.0, "3d": 8.0}.get(case["op"], 10.0)
    return {"bytes": (16.0 + data) * n, "flops": (apply + 10.0) * n * _iterations(case, dims)}


def _sine_solve(b, dims):
    """A^-1 b of the constant stencil through its sine eigenvectors."""
    dims = list(dims) + [1] * (3 - len(dims))
    S, lam = [], []
    for d in dims:
        k = torch.arange(1, d + 1, dtype=torch.float64, device=b.device)
        S.append(torch.sin(math.pi * torch.outer(k, k) / (d + 1)) * math.sqrt(2.0 / (d + 1)))
        lam.append(4.0 * torch.sin(math.pi * k / (2 * (d + 1))) ** 2)
    nx, ny, nz = dims

    def transform(v):
        v = (v.reshape(nz * ny, nx) @ S[0]).reshape(nz, ny, nx)
        v = v.transpose(1, 2).reshape(nz * nx, ny) @ S[1]
        v = v.reshape(nz, nx, ny).transpose(1, 2)
        return S[2] @ v.reshape(nz, ny * nx) if nz > 1 else v

    scale = lam[1][:, None] + lam[0][None, :]
    if nz > 1:
        scale = scale[None] + lam[2][:, None, None]
    return transform(transform(b).reshape(scale.shape) / scale).reshape(-1)


def _stencil(dims):
    shape = tuple(reversed(dims))

    def apply(v):
        v = v.reshape(shape)
        w = 2.0 * len(dims) * v
        for axis, d in enumerate(shape):
            lo, hi = v.narrow(axis, 0, d - 1), v.narrow(axis, 1, d - 1)
            w.narrow(axis, 0, d - 1).sub_(hi)
            w.narrow(axis, 1, d - 1).sub_(lo)
        return w.reshape(-1)

    return apply


def _edge_operator(cx, cy):
    """The Jacobi-scaled operator D^-1/2 A D^-1/2 and D^-1/2."""
    d = _diagonal(cx, cy)
    dis = d.rsqrt()
    ex = cx[:, 1:-1] * dis[:, :-1] * dis[:, 1:]
    ey = cy[1:-1] * dis[:-1] * dis[1:]

    def apply(v):
        v = v.reshape(d.shape)
        w = v.clone()
        w[:, :-1] -= ex * v[:, 1:]
        w[:, 1:] -= ex * v[:, :-1]
        w[:-1] -= ey * v[1:]
        w[1:] -= ey * v[:-1]
        return w.reshape(-1)

    return apply, dis.reshape(-1)


def _cg(apply, b, tol, maxit):
    """Textbook CG from x0 = 0: the iterate whose ||r|| is first below tol ||b||, or the
    maxit-th.  The stop is looked for every 25 iterations when there is no budget to keep."""
    x, r = torch.zeros_like(b), b.clone()
    p, rho = r.clone(), torch.dot(r, r)
    stop = float(rho.sqrt()) * tol
    every = 1 if maxit < 100000 else 25
    for k in range(maxit):
        q = apply(p)
        alpha = rho / torch.dot(p, q)
        x.addcmul_(p, alpha)
        r.addcmul_(q, -alpha)
        new = torch.dot(r, r)
        if k % every == every - 1 and float(new.sqrt()) < stop:
            break
        p.mul_(new / rho).add_(r)
        rho = new
    return x


def exact(case, seed):
    if case["op"] == "serve":
        out = []
        for k, (nx, ny) in enumerate(_sides(case)):
            A, dis = _edge_operator(*_edges(nx, ny, seed * 1000 + k))
            out.append(dis * _cg(A, dis * _rhs(nx * ny, seed * 1000 + k), 1e-13, 100000))
        return out
    dims = _dims(case)
    b = _rhs(math.prod(dims), seed)
    if case["op"] in ("2d", "3d"):
        if case["maxit"] < 100000:
            return _cg(_stencil(dims), b, case["tol"], case["maxit"])
        return _sine_solve(b, dims)
    A, dis = _edge_operator(*_edges(*dims, seed))
    if case["maxit"] < 100000:
        return dis * _cg(A, dis * b, case["tol"], case["maxit"])
    return dis * _cg(A, dis * b, 1e-13, 100000)
