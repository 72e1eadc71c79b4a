"""The work that a program does with this solver, as cases whose time can be measured.

A case is a dict of plain values: ``path`` names the entry point, the rest its sizes and
options.  The ranges are those of the lattice and grid problems this repository's
workloads, tests and benchmark use: staggered lattices from 4^4 to 32^3 x 64, 2-D and 3-D
grids of up to 10^6 points, 4 to 16 shifts, one to four right-hand sides.

Inputs are made on the GPU from the seed alone: Haar SU(3) links (unit links multiplied at
random, the stand-in for gauge configurations used throughout), complex Gaussian
right-hand sides, log-spaced shifts.
"""
import math

import torch

from paper_1102_2143_amd import Operator
from paper_1102_2143_amd.api import solve_batched
from paper_1102_2143_amd.autograd import multishift_solve

DEV = "cuda:0"
C128 = torch.complex128


# ---- inputs ----------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + stream)
    return g


def _gauss(g, *shape):
    z = torch.randn(*shape, 2, generator=g, device=DEV, dtype=torch.float64)
    return torch.view_as_complex(z) * math.sqrt(0.5)


def _extents(text):
    return tuple(int(v) for v in text.split("x"))


def _links(g, dims):
    """Haar SU(3) links (4, V, 3, 3): two orthonormal random rows, the third their
    conjugated cross product."""
    vol = math.prod(dims)
    z = _gauss(g, 4 * vol, 2, 3)
    u = z[:, 0] / z[:, 0].abs().square().sum(1, keepdim=True).sqrt()
    v = z[:, 1]
    for _ in range(2):
        v = v - (u.conj() * v).sum(1, keepdim=True) * u
    v = v / v.abs().square().sum(1, keepdim=True).sqrt()
    w = torch.linalg.cross(u, v).conj()
    return torch.stack([u, v, w], 1).reshape(4, vol, 3, 3)


def _shifts(case):
    return torch.logspace(math.log10(case["lo"]), math.log10(case["hi"]), case["ns"],
                          dtype=torch.float64).tolist()


def _lattice(dims):
    """Per direction: the forward and backward neighbour of every site and eta_mu / 2."""
    vol = math.prod(dims)
    s = torch.arange(vol, device=DEV)
    stride, run, out = 1, torch.zeros_like(s), []
    for L in dims:
        c = (s // stride) % L
        fwd = s + torch.where(c == L - 1, -(L - 1) * stride, stride)
        bwd = s + torch.where(c == 0, (L - 1) * stride, -stride)
        out.append((fwd, bwd, 0.5 - (run % 2).double()))
        run, stride = run + c, stride * L
    return out


def _staggered_csr(links, dims, mass):
    """CSR of M = mass + D for the given links: 25 sorted entries per row."""
    vol = math.prod(dims)
    site = torch.arange(vol, device=DEV)
    col3 = torch.arange(3, device=DEV)
    cols = [(3 * site[:, None] + col3)[:, :, None]]
    vals = [torch.full((vol, 3, 1), mass, device=DEV, dtype=C128)]
    for (fwd, bwd, half), u in zip(_lattice(dims), links):
        w = half[:, None, None] * u
        for nb, m in ((fwd, w), (bwd, -w[bwd].mH)):
            cols.append((3 * nb[:, None, None] + col3).expand(vol, 3, 3))
            vals.append(m)
    cols, order = torch.cat(cols, 2).sort(2)
    vals = torch.cat(vals, 2).gather(2, order)
    rowptr = torch.arange(0, 75 * vol + 1, 25, device=DEV)
    return rowptr, cols.reshape(-1).int(), vals.reshape(-1)


def _grid(ext, diag, off):
    """CSR of a Dirichlet grid operator: `diag` (n,) on the diagonal and, for direction mu,
    off[mu] = (value towards the lower, towards the upper neighbour)."""
    n = math.prod(ext)
    s = torch.arange(n, device=DEV)
    stride, low, high = 1, [], []
    for L, (lo, hi) in zip(ext, off):
        c = (s // stride) % L
        low.insert(0, (s - stride, c > 0, lo))
        high.append((s + stride, c < L - 1, hi))
        stride *= L
    cand = [(c, ok, torch.full((n,), v, device=DEV, dtype=C128)) for c, ok, v in low]
    cand.append((s, torch.ones_like(s, dtype=torch.bool), diag.to(C128)))
    cand += [(c, ok, torch.full((n,), v, device=DEV, dtype=C128)) for c, ok, v in high]
    ok = torch.stack([c[1] for c in cand], 1)
    cols = torch.stack([c[0] for c in cand], 1)[ok].int()
    vals = torch.stack([c[2] for c in cand], 1)[ok]
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = ok.sum(1).cumsum(0)
    return rowptr, cols, vals


def _grid_case(g, case):
    """(extents, diagonal, off-diagonal values) of the grid operator of a case."""
    ext = _extents(case["dims"])
    n = math.prod(ext)
    if case["path"] == "solve_real":      # the 2-D five-point Poisson matrix
        return ext, torch.full((n,), 4.0, device=DEV, dtype=torch.float64), [(-1.0, -1.0)] * 2
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    if case["path"] == "solve_bicgstab":  # convection and diffusion: not Hermitian
        return ext, 6.05 + 0.95 * u, [(-1.0 - f, -1.0 + f) for f in (0.3, 0.2, 0.1)]
    return ext, 6.01 + 0.99 * u, [(-1.0, -1.0)] * 3


BATCH = ("4x4x4x4", "6x6x6x6", "8x8x8x8", "12x12x12x12")


def _batch(case):
    """(kind, extents) of each system of a batch: lattices of four sizes in turn, then
    grids, as the batch workload mixes them."""
    k = ["mhm"] * case["lattices"] + ["herm"] * case["grids"]
    return [(kind, BATCH[i % 4] if kind == "mhm" else case["dims"]) for i, kind in enumerate(k)]


def _batch_system(seed, i, kind, dims, case):
    g = _gen(seed, 100 + i)
    ext = _extents(dims)
    n = math.prod(ext) * (3 if kind == "mhm" else 1)
    if kind == "mhm":
        a = _links(g, ext)
    else:
        a = 6.01 + 0.99 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    return ext, n, a, _gauss(g, case["nrhs"], n)


# ---- the cases --------------------------------------------------------------------------
def listed():
    return [
        # one product with A on the smallest lattice: latency of a call
        dict(name="apply-4^4", path="apply", dims="4x4x4x4", mass=0.1),
        # the product alone at the largest lattice: heat baths, energies, residual checks
        dict(name="apply-32^3x64", path="apply", dims="32x32x32x64", mass=0.02),
        # the smallest solve, launch bound: tests, tuning runs, coarse ensembles
        dict(name="solve-links-4^4-fp64", path="solve_links", dims="4x4x4x4", mass=0.1, ns=8,
             lo=1e-4, hi=1.0, prec="fp64", tol=1e-10),
        # molecular dynamics: new links, then the family of solves on them; a ragged lattice
        dict(name="md-12x10x14x18-fp64", path="md", dims="12x10x14x18", mass=0.05, ns=12,
             lo=1e-5, hi=10.0, prec="fp64", tol=1e-10),
        # an ordinary lattice handed over as a stored matrix, in mixed precision
        dict(name="solve-csr-16^4-mixed", path="solve_csr", dims="16x16x16x16", mass=0.05, ns=12,
             lo=1e-5, hi=10.0, prec="mixed", tol=1e-10),
        # the largest solve of the benchmark
        dict(name="solve-links-32^3x64-mixed", path="solve_links", dims="32x32x32x64", mass=0.02,
             ns=16, lo=1e-6, hi=10.0, prec="mixed", tol=1e-10),
        # a Hermitian matrix given directly, on a ragged grid
        dict(name="solve-herm-61x50x45-fp64", path="solve_herm", dims="61x50x45", ns=10, lo=1e-4,
             hi=1.0, prec="fp64", tol=1e-10),
        # the 2-D Poisson benchmark of the method's paper, real arithmetic
        dict(name="solve-real-1000^2-fp64", path="solve_real", dims="1000x1000", ns=15, lo=1e-3,
             hi=1.0, prec="fp64", tol=1e-5),
        # many small systems at once
        dict(name="batch-64-mixed", path="batch", lattices=48, grids=16, dims="32x32x32", mass=0.1,
             ns=10, lo=1e-4, hi=1.0, nrhs=4, prec="mixed", tol=1e-10),
        # a training step: forward and backward, gradients of the matrix and of b
        dict(name="grad-16^4-fp64", path="grad", dims="16x16x16x16", mass=0.1, ns=10, lo=1e-4,
             hi=1.0, prec="fp64", tol=1e-10),
        # a right-hand side for each shift
        dict(name="multi-rhs-16^4-fp64", path="multi_rhs", dims="16x16x16x16", mass=0.1, ns=10,
             lo=1e-4, hi=1.0, prec="fp64", tol=1e-10),
        # a matrix that is not Hermitian
        dict(name="bicgstab-64x48x50", path="solve_bicgstab", dims="64x48x50", ns=8, lo=1e-3,
             hi=1.0, prec="fp64", tol=1e-10),
    ]


def _some_lattice(rng, least, most):
    """Extents with a volume about log-uniform in [least, most], odd ones among them."""
    vol = math.exp(rng.uniform(math.log(least), math.log(most)))
    side = vol ** 0.25
    ext = [max(3, round(side * math.exp(rng.uniform(-0.25, 0.25)))) for _ in range(3)]
    if rng.random() < 0.6:
        ext = [e + e % 2 for e in ext]
    last = max(3, round(vol / math.prod(ext)))
    return "x".join(str(e) for e in ext + [last + last % 2 if rng.random() < 0.6 else last])


def _some_grid(rng, d, least, most):
    n = math.exp(rng.uniform(math.log(least), math.log(most)))
    ext = [max(3, round(n ** (1 / d) * math.exp(rng.uniform(-0.2, 0.2)))) for _ in range(d - 1)]
    return "x".join(str(e) for e in ext + [max(3, round(n / math.prod(ext)))])


def draw(rng):
    path = rng.choice(["apply", "solve_links", "solve_links", "md", "solve_csr", "solve_herm",
                       "solve_real", "batch", "grad", "multi_rhs", "solve_bicgstab"])
    c = dict(path=path)
    if path == "apply":
        return dict(c, dims=_some_lattice(rng, 256, 2 ** 21), mass=0.05)
    c.update(ns=rng.randint(4, 14), lo=rng.choice([1e-4, 1e-3]), hi=rng.choice([1.0, 10.0]))
    if path in ("solve_links", "md", "solve_csr"):
        most = 400_000 if path == "solve_links" else 150_000
        prec = rng.choice(["fp64", "mixed"])
        return dict(c, dims=_some_lattice(rng, 256, most), mass=rng.choice([0.05, 0.1]), prec=prec,
                    tol=1e-10)
    if path == "solve_real":
        return dict(c, dims=_some_grid(rng, 2, 2_000, 1_000_000), lo=1e-3, prec="fp64", tol=1e-5)
    if path == "solve_herm":
        return dict(c, dims=_some_grid(rng, 3, 1_000, 300_000), prec="fp64", tol=1e-10)
    if path == "solve_bicgstab":
        return dict(c, dims=_some_grid(rng, 3, 1_000, 300_000), ns=rng.randint(4, 10), lo=1e-3,
                    prec="fp64", tol=1e-10)
    if path == "batch":
        return dict(c, lattices=rng.randint(2, 16), grids=rng.randint(0, 8),
                    dims=_some_grid(rng, 3, 2_000, 40_000), mass=0.1, ns=rng.randint(4, 10),
                    nrhs=rng.choice([1, 2, 4]), prec=rng.choice(["fp64", "mixed"]), tol=1e-10)
    return dict(c, dims=_some_lattice(rng, 256, 80_000), mass=0.1, ns=rng.randint(4, 12),
                hi=1.0, prec="fp64", tol=1e-10)


# ---- one pass ---------------------------------------------------------------------------
def prepare(case, seed):
    path, g = case["path"], _gen(seed, 0)
    if path == "batch":
        ops, bs = [], []
        for i, (kind, dims) in enumerate(_batch(case)):
            ext, n, a, b = _batch_system(seed, i, kind, dims, case)
            if kind == "mhm":
                op = Operator.staggered(a, ext, case["mass"], device=DEV)
            else:
                op = Operator(*_grid(ext, a, [(-1.0, -1.0)] * 3), n, kind="herm", device=DEV)
            op.set_shifts(_shifts(case))
            ops.append(op)
            bs.append(b)
        return dict(case=case, ops=ops, bs=bs)
    st = dict(case=case)
    if path in ("solve_herm", "solve_real", "solve_bicgstab"):
        ext, diag, off = _grid_case(g, case)
        n = math.prod(ext)
        st["op"] = Operator(*_grid(ext, diag, off), n, device=DEV,
                            kind="general" if path == "solve_bicgstab" else "herm")
        if path == "solve_real":
            st["b"] = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
        else:
            st["b"] = _gauss(g, n)
        st["op"].set_shifts(_shifts(case))
        return st
    dims = _extents(case["dims"])
    n = 3 * math.prod(dims)
    links = _links(g, dims)
    if path in ("solve_csr", "grad"):
        rowptr, col, vals = _staggered_csr(links, dims, case["mass"])
        st["op"] = Operator(rowptr, col, vals, n, kind="mhm", device=DEV)
        if path == "grad":
            st["vals"] = vals.requires_grad_()
            st["target"] = _gauss(_gen(seed, 1), case["ns"], n)
    else:
        st["op"] = Operator.staggered(links, dims, case["mass"], device=DEV)
    if path == "md":
        st["links"] = _links(_gen(seed, 2), dims)  # the next step's links
    if path != "apply":
        st["op"].set_shifts(_shifts(case))
    st["b"] = _gauss(_gen(seed, 3), case["ns"], n) if path == "multi_rhs" else _gauss(_gen(seed, 3), n)
    if path == "grad":
        st["b"].requires_grad_()
    return st


def run(state):
    case = state["case"]
    path = case["path"]
    if path == "apply":
        return state["op"].apply(state["b"])
    kw = dict(tol=case["tol"], prec=case["prec"])
    if path == "batch":
        return solve_batched(state["ops"], state["bs"], **kw)[0]
    op, b = state["op"], state["b"]
    if path == "md":
        op.update_links(state["links"])
    if path == "grad":
        vals = state["vals"]
        vals.grad = b.grad = None
        x = multishift_solve(vals, b, op, **kw)
        loss = (x - state["target"]).abs().square().sum()
        loss.backward()
        return dict(x=x.detach(), grad_b=b.grad, grad_vals=vals.grad)
    call = {"solve_real": op.solve_real, "solve_bicgstab": op.solve_bicgstab,
            "multi_rhs": op.solve_multi_rhs}.get(path, op.solve)
    return call(b, **kw)[0]


# ---- what a pass cannot do without --------------------------------------------------------
def _iterations(case, least, most):
    """Steps of CG to the tolerance on a spectrum [least, most]: sqrt(condition) / 2 times
    the logarithm, somewhat less on these spectra."""
    return 0.45 * math.sqrt(most / least) * math.log(2.0 / case["tol"])


def _one(kind, n, case, nrhs=1, steps=None):
    """Bytes and operations of one family: per step the operator, the driving vectors and
    the shifted vectors once, at the width of the arithmetic (the mean of both in mixed
    precision); the shifts beyond the driving one leave early, a third of the steps on
    average."""
    real = case["path"] == "solve_real"
    w = (8 if real else 16) * (0.75 if case["prec"] == "mixed" else 1.0)
    if kind == "links":      # four links of two rows a site for both halves, each half
        mat, ops = 2 * 8 * w, 2 * 200
    elif kind == "mhm":
        mat, ops = 2 * 25 * (w + 2), 2 * 200
    else:
        mat, ops = 7 * (w + 2), 56
    if steps is None:
        if kind in ("links", "mhm"):
            steps = _iterations(case, case["mass"] ** 2 + case["lo"], 3.5)
        elif len(case["dims"].split("x")) == 2:
            steps = _iterations(case, case["lo"], 8.0)
        else:
            steps = _iterations(case, 0.1, 12.0)
    vec = 10 * w + (case["ns"] - 1) / 3 * 4 * w / 8
    lin = 10 * 8 + (case["ns"] - 1) / 3 * 32
    return steps * n * (mat + nrhs * vec), steps * n * nrhs * (ops + lin)


def work(case):
    path = case["path"]
    if path == "batch":
        tot = [0.0, 0.0]
        for kind, dims in _batch(case):
            n = math.prod(_extents(dims)) * (3 if kind == "mhm" else 1)
            for i, v in enumerate(_one(kind, n, dict(case, dims=dims), case["nrhs"])):
                tot[i] += v
        return dict(bytes=tot[0], flops=tot[1])
    n = math.prod(_extents(case["dims"]))
    if path in ("solve_herm", "solve_real", "solve_bicgstab"):
        by, fl = _one("grid", n, case)
        k = 2 if path == "solve_bicgstab" else 1  # two products a step, half the steps
        return dict(bytes=k * by, flops=k * fl)
    n *= 3
    if path == "apply":
        return dict(bytes=n * 16 * (8 + 2), flops=n * 400)
    by, fl = _one("mhm" if path in ("solve_csr", "grad") else "links", n, case)
    if path in ("grad", "multi_rhs"):  # the systems one by one, the operator once
        b2, f2 = _one("mhm" if path == "grad" else "links", n, dict(case, ns=1), case["ns"])
        by, fl = (by + b2, fl + f2) if path == "grad" else (b2, f2)
    return dict(bytes=by, flops=fl)


# ---- the values in 64 bits ----------------------------------------------------------------
def _hop(links, dims):
    """v (k, V, 3) -> D v, for links (4, V, 3, 3)."""
    legs = []
    for (fwd, bwd, half), u in zip(_lattice(dims), links):
        w = half[:, None, None] * u
        legs += [(fwd, w), (bwd, -w[bwd].mH)]

    def d(v):
        out = torch.zeros_like(v)
        for nb, w in legs:
            h = v[:, nb]
            for j in range(3):
                out += w[:, :, j] * h[:, :, j, None]
        return out
    return d


def _lattice_op(links, dims, mass):
    """(k, n) -> M^H M and M."""
    d, vol = _hop(links, dims), math.prod(dims)

    def m(v):
        v = v.reshape(-1, vol, 3)
        return (mass * v + d(v)).reshape(v.shape[0], -1)

    def a(v):
        t = m(v).reshape(-1, vol, 3)
        return (mass * t - d(t)).reshape(t.shape[0], -1)
    return a, m


def _grid_op(ext, diag, off):
    def a(v):
        g = v.reshape(-1, *reversed(ext))
        out = diag.reshape(tuple(reversed(ext))) * g
        for mu, (lo, hi) in enumerate(off):
            ax = g.dim() - 1 - mu
            L = ext[mu]
            out.narrow(ax, 1, L - 1).add_(lo * g.narrow(ax, 0, L - 1))
            out.narrow(ax, 0, L - 1).add_(hi * g.narrow(ax, 1, L - 1))
        return out.reshape(v.shape)
    return a


def _dot(u, v):
    return (u.conj() * v).sum(1, keepdim=True)


def _cg(apply, b, sig):
    """(A + sig_k) x_k = b_k by plain CG, each to rounding; one pass of correction."""
    s = torch.tensor(sig, device=DEV, dtype=torch.float64)[:, None]
    x = torch.zeros_like(b)
    target = 1e-30 * _dot(b, b).real
    for _ in range(2):
        r = b - apply(x) - s * x
        p, rr = r.clone(), _dot(r, r).real
        start = rr.clone()
        for it in range(6000):
            if it % 25 == 0 and bool(((rr <= target) | (rr <= 1e-26 * start)).all()):
                break
            q = apply(p) + s * p
            a = rr / _dot(p, q).real.clamp_min(1e-300)
            x += a * p
            r -= a * q
            new = _dot(r, r).real
            p = r + (new / rr.clamp_min(1e-300)) * p
            rr = new
    return x


def _bicgstab(apply, b, sig):
    s = torch.tensor(sig, device=DEV, dtype=torch.float64)[:, None]
    x = torch.zeros_like(b)
    for _ in range(3):
        r = b - apply(x) - s * x
        w, p, rho = r.clone(), r.clone(), _dot(r, r)
        goal = 1e-24 * _dot(r, r).real
        for it in range(3000):
            if it % 10 == 0 and bool((_dot(r, r).real <= goal).all()):
                break
            v = apply(p) + s * p
            alpha = rho / _dot(w, v)
            h = r - alpha * v
            t = apply(h) + s * h
            om = _dot(t, h) / _dot(t, t)
            live = _dot(r, r).real > goal
            x = torch.where(live, x + alpha * p + om * h, x)
            rn = h - om * t
            new = _dot(w, rn)
            p = torch.where(live, rn + (new / rho) * (alpha / om) * (p - om * v), p)
            r, rho = torch.where(live, rn, r), torch.where(live, new, rho)
    return x


def exact(case, seed):
    path, g = case["path"], _gen(seed, 0)
    if path == "batch":
        return _exact_batch(case, seed)
    ext = _extents(case["dims"])
    if path == "solve_real":  # sines diagonalise the matrix
        _grid_case(g, case)
        nx, ny = ext
        b = torch.randn(nx * ny, generator=g, device=DEV, dtype=torch.float64)
        s, lam = [], []
        for L in ext:
            k = torch.arange(1, L + 1, device=DEV, dtype=torch.float64)
            s.append(math.sqrt(2 / (L + 1)) * torch.sin(math.pi / (L + 1) * ((k[:, None] * k) % (2 * (L + 1)))))
            lam.append(2 - 2 * torch.cos(math.pi * k / (L + 1)))
        f = s[1] @ b.reshape(ny, nx) @ s[0]
        ev = lam[1][:, None] + lam[0]
        return torch.stack([(s[1] @ (f / (ev + z)) @ s[0]).reshape(-1) for z in _shifts(case)])
    if path in ("solve_herm", "solve_bicgstab"):
        ext, diag, off = _grid_case(g, case)
        b = _gauss(g, math.prod(ext)).expand(case["ns"], -1).contiguous()
        solver = _cg if path == "solve_herm" else _bicgstab
        return solver(_grid_op(ext, diag, off), b, _shifts(case))
    n = 3 * math.prod(ext)
    links = _links(g, ext)
    if path == "md":
        links = _links(_gen(seed, 2), ext)
    a, m = _lattice_op(links, ext, case["mass"])
    if path == "apply":
        return a(_gauss(_gen(seed, 3), n)[None])[0]
    if n > 1_000_000:
        return None  # minutes in plain torch
    ns = case["ns"]
    if path == "multi_rhs":
        return _cg(a, _gauss(_gen(seed, 3), ns, n), _shifts(case))
    x = _cg(a, _gauss(_gen(seed, 3), n).expand(ns, -1).contiguous(), _shifts(case))
    if path != "grad":
        return x
    y = _cg(a, 2 * (x - _gauss(_gen(seed, 1), ns, n)), _shifts(case))
    _, col, _ = _staggered_csr(links, ext, case["mass"])
    col = col.long().reshape(n, 25)
    mx, my = m(x), m(y)
    gv = torch.zeros(n, 25, device=DEV, dtype=C128)
    for k in range(ns):
        gv -= my[k][:, None] * x[k].conj()[col] + mx[k][:, None] * y[k].conj()[col]
    return dict(x=x, grad_b=y.sum(0), grad_vals=gv.reshape(-1))


def _exact_batch(case, seed):
    """Systems of one kind and size together: the batch as one block-diagonal system."""
    ns, nrhs, sig = case["ns"], case["nrhs"], _shifts(case)
    if case["lattices"] + case["grids"] > 24:
        return None  # over the time that is wanted
    out = []
    for i, (kind, dims) in enumerate(_batch(case)):
        ext, n, a, b = _batch_system(seed, i, kind, dims, case)
        op = _lattice_op(a, ext, case["mass"])[0] if kind == "mhm" else _grid_op(ext, a, [(-1.0, -1.0)] * 3)
        f = b[:, None].expand(nrhs, ns, n).reshape(nrhs * ns, n).contiguous()
        out.append(_cg(op, f, sig * nrhs).reshape(nrhs, ns, n))
    return out
