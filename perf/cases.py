"""Performance cases: the work a program that uses this library has it do.

Every case is one pass through the public entry points of
``paper_2606_09001_amd.solver`` on systems built on the device: handles kept
across solves, one-shot solves, value updates followed by a solve, blocks of
right-hand sides, same-pattern systems, the differentiable solve, the
nonsymmetric solver with its adjoint, plain CG and the V-cycle as an operator.
"""
import math

import torch

from paper_2606_09001_amd import matrices as M
from paper_2606_09001_amd.solver import AmgHierarchy, amg_solve, finalize, solve

DEV = "cuda"
F64 = torch.float64


# ------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest call: a 1,024-unknown solve inside another program's loop
        dict(name="poisson2d-32", kind="solve", matrix="poisson", d=2, N=32, prec="fp64", tol=1e-10),
        # a 2D system of ordinary size with a ragged edge (181^2 = 32,761 rows): bound by launches
        dict(name="diffusion2d-181", kind="solve", matrix="diffusion", d=2, N=181, prec="fp64", tol=1e-10),
        # the benchmark: constant-coefficient 3D Poisson, FP64, hierarchy kept
        dict(name="poisson3d-128", kind="solve", matrix="poisson", d=3, N=128, prec="fp64", tol=1e-8),
        # the largest single system: lognormal diffusion, mixed precision, hierarchy kept
        dict(name="diffusion3d-192-mixed", kind="solve", matrix="diffusion", d=3, N=192, prec="fp32", tol=1e-8),
        # one step of learning a coefficient field: new values, forward solve, adjoint, pattern gradient
        dict(name="train2d-512", kind="train", d=2, N=512, prec="fp64", tol=1e-10),
        # many right-hand sides of one matrix (load cases, probing, uncertainty samples)
        dict(name="rhs32-poisson3d-128", kind="solve", matrix="poisson", d=3, N=128, prec="fp64", tol=1e-8, cols=32),
        # a step of 64 coefficient samples at once: new values of every system, mixed-precision solve
        dict(name="systems64-diffusion3d-64", kind="systems", d=3, N=64, prec="fp32", tol=1e-8, cols=64),
        # a program that meets a matrix once: cold setup and one solve
        dict(name="oneshot-diffusion3d-100", kind="oneshot", d=3, N=100, prec="fp64", tol=1e-8),
        # a time step of a nonlinear problem: new values on the known pattern, then a solve
        dict(name="step-diffusion3d-128", kind="step", d=3, N=128, prec="fp64", tol=1e-8),
        # convection-diffusion with BiCGSTAB: forward, adjoint and pattern gradient on kept hierarchies
        dict(name="convection3d-96", kind="convection", d=3, N=96, prec="fp64", tol=1e-12, speed=300.0),
        # unpreconditioned CG on a large well-conditioned tridiagonal system
        dict(name="plain-tridiag-1e7", kind="plain", N=10_000_000, tol=1e-10),
        # the V-cycle as an operator for another Krylov loop, odd grid (FP64: a mixed cycle returns its FP32
        # rounding in FP64 values, which says nothing at the accuracy FP64 values are compared to)
        dict(name="vcycle-diffusion3d-111", kind="vcycle", d=3, N=111, prec="fp64"),
    ]


def _size(rng, lo, hi):
    """Grid points per axis, spread over the logarithm; as often odd as even."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "train", "rhs", "systems", "oneshot", "step", "convection", "plain",
                       "vcycle"])
    d = rng.choice([2, 3])
    prec = rng.choice(["fp64", "fp64", "fp32"])
    tol = rng.choice([1e-8, 1e-10])
    matrix = rng.choice(["poisson", "diffusion"])
    if kind == "solve":
        N = _size(rng, 20, 900) if d == 2 else _size(rng, 10, 170)
        return dict(kind="solve", matrix=matrix, d=d, N=N, prec=prec, tol=tol)
    if kind == "train":
        return dict(kind="train", d=2, N=_size(rng, 48, 640), prec="fp64", tol=1e-10)
    if kind == "rhs":
        N = _size(rng, 40, 400) if d == 2 else _size(rng, 12, 96)
        return dict(kind="solve", matrix=matrix, d=d, N=N, prec=prec, tol=tol, cols=rng.randint(2, 40))
    if kind == "systems":
        N = _size(rng, 40, 250) if d == 2 else _size(rng, 12, 56)
        return dict(kind="systems", d=d, N=N, prec=prec, tol=tol, cols=rng.randint(2, 64))
    if kind == "oneshot":
        return dict(kind="oneshot", d=d, N=_size(rng, 40, 700) if d == 2 else _size(rng, 12, 110), prec=prec, tol=tol)
    if kind == "step":
        return dict(kind="step", d=d, N=_size(rng, 40, 700) if d == 2 else _size(rng, 12, 150), prec=prec, tol=tol)
    if kind == "convection":
        N = _size(rng, 40, 250) if d == 2 else _size(rng, 14, 96)
        return dict(kind="convection", d=d, N=N, prec="fp64", tol=1e-12, speed=float(rng.randint(50, 300)))
    if kind == "plain":
        return dict(kind="plain", N=_size(rng, 20_000, 10_000_000), tol=1e-10)
    return dict(kind="vcycle", d=d, N=_size(rng, 30, 900) if d == 2 else _size(rng, 12, 160), prec="fp64")


# ------------------------------------------------- matrices on the device

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(shape, g):
    return torch.randn(shape, generator=g, device=DEV, dtype=F64)


def _coords(N, d):
    """Grid index along each axis (axis 0 = x, fastest) of every unknown."""
    i = torch.arange(N ** d, device=DEV)
    return [(i // N ** a) % N for a in range(d)]


def _offsets(N, d):
    """(column offset, axis, side) of the stencil in ascending column order."""
    return ([(-N ** a, a, -1) for a in reversed(range(d))] + [(0, -1, 0)] + [(N ** a, a, 1) for a in range(d)])


def _present(N, d):
    c = _coords(N, d)
    cols = []
    for _, a, side in _offsets(N, d):
        cols.append(torch.ones(N ** d, dtype=torch.bool, device=DEV) if side == 0 else
                    c[a] > 0 if side < 0 else c[a] < N - 1)
    return torch.stack(cols, dim=1)


def _pattern(N, d):
    """CSR row pointers and columns of the (2d+1)-point stencil, and its mask."""
    mask = _present(N, d)
    rp = torch.zeros(N ** d + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(mask.sum(dim=1), dim=0)
    off = torch.tensor([o for o, _, _ in _offsets(N, d)], device=DEV)
    col = torch.arange(N ** d, device=DEV)[:, None] + off[None, :]
    return rp, col[mask].to(torch.int32), mask


def _lognormal(N, d, g):
    """exp of a Gaussian field with a squared-exponential covariance of length
    0.1: a sum of cosines with normally distributed wave numbers."""
    modes = 32
    k = (_normal((modes, d), g) / 0.1).tolist()
    ph = (torch.rand(modes, generator=g, device=DEV, dtype=F64) * (2 * math.pi)).tolist()
    ax = (torch.arange(N, device=DEV, dtype=F64) + 1) / (N + 1)
    grids = [ax.view([N if a == d - 1 - b else 1 for a in range(d)]) for b in range(d)]
    f = torch.zeros((N,) * d, device=DEV, dtype=F64)
    for m in range(modes):
        f = f + torch.cos(sum(k[m][a] * grids[a] for a in range(d)) + ph[m])
    return torch.exp(f * math.sqrt(2.0 / modes))


def _diffusion_values(k, mask):
    """Values of -div(k grad u) with harmonic-mean faces on the stencil's pattern."""
    d, N = k.dim(), k.shape[0]
    lo, hi = [], []
    for a in range(d):
        ax = d - 1 - a
        p, q = k.narrow(ax, 0, N - 1), k.narrow(ax, 1, N - 1)
        f = ((2.0 * p) * q) / (p + q)
        lo.append(torch.cat([k.narrow(ax, 0, 1), f], dim=ax).reshape(-1))
        hi.append(torch.cat([f, k.narrow(ax, N - 1, 1)], dim=ax).reshape(-1))
    diag = torch.zeros(N ** d, dtype=k.dtype, device=k.device)
    for a in range(d):
        diag = diag + lo[a]
        diag = diag + hi[a]
    vals = [diag if side == 0 else -lo[a] if side < 0 else -hi[a] for _, a, side in _offsets(N, d)]
    return torch.stack(vals, dim=1)[mask]


def _poisson_values(N, d, mask):
    row = torch.tensor([2.0 * d if side == 0 else -1.0 for _, _, side in _offsets(N, d)], dtype=F64, device=DEV)
    return row[None, :].expand(N ** d, -1)[mask]


def _convection_values(N, d, speed, mask):
    """Upwind convection-diffusion in a recirculating flow, scaled by h^2."""
    h = 1.0 / (N + 1)
    x = [(c.to(F64) + 1) * h for c in _coords(N, d)[:2]]
    w = [speed * torch.sin(math.pi * x[0]) * torch.cos(math.pi * x[1]),
         -speed * torch.cos(math.pi * x[0]) * torch.sin(math.pi * x[1])] + [torch.zeros_like(x[0])] * (d - 2)
    vals = []
    for _, a, side in _offsets(N, d):
        if side == 0:
            vals.append(2.0 * d + h * sum(wa.abs() for wa in w))
        else:
            vals.append(-1.0 - h * torch.clamp(w[a] if side < 0 else -w[a], min=0.0))
    return torch.stack(vals, dim=1)[mask]


def _tridiagonal(n):
    """tridiag(-1, 2.5, -1)"""
    rp = torch.arange(n + 1, device=DEV) * 3 - 1
    rp[0], rp[n] = 0, 3 * n - 2
    k = torch.arange(3 * n - 2, device=DEV) + 1
    col = (k // 3 + k % 3 - 1).to(torch.int32)
    val = torch.where(k % 3 == 1, 2.5, -1.0).to(F64)
    return rp.to(torch.int32), col, val


def _matrix(c, g):
    N, d = c["N"], c["d"]
    rp, col, mask = _pattern(N, d)
    if c["kind"] == "convection":
        return rp, col, _convection_values(N, d, c["speed"], mask)
    if c.get("matrix") == "poisson":
        return rp, col, _poisson_values(N, d, mask)
    if c["kind"] == "systems":
        v = torch.empty(len(col), c["cols"], dtype=F64, device=DEV)
        for s in range(c["cols"]):
            v[:, s] = _diffusion_values(_lognormal(N, d, g), mask)
        return rp, col, v
    return rp, col, _diffusion_values(_lognormal(N, d, g), mask)


def _inputs(c, seed):
    """The case's system and vectors, from the seed alone."""
    g = _gen(seed)
    if c["kind"] == "plain":
        A = _tridiagonal(c["N"])
        return dict(A=A, b=_normal((c["N"],), g))
    if c["kind"] == "train":
        N, d = c["N"], c["d"]
        rp, col, mask = _pattern(N, d)
        theta = torch.log(_lognormal(N, d, g))
        ax = torch.sin(math.pi * (torch.arange(N, device=DEV, dtype=F64) + 1) / (N + 1))
        target = 0.05 * N * N * (ax[:, None] * ax[None, :]).reshape(-1)
        return dict(A=(rp, col, mask), theta=theta, b=torch.ones(N ** d, dtype=F64, device=DEV), target=target)
    A = _matrix(c, g)
    n = len(A[0]) - 1
    s = dict(A=A, b=_normal((n, c["cols"]) if "cols" in c else (n,), g))
    if c["kind"] == "convection":
        s["g"] = _normal((n,), g)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    s["kind"], s["tol"] = kind, case.get("tol")
    if kind == "train":
        s["kw"] = dict(vcycle_prec=case["prec"])
    elif kind == "convection":
        s["H"] = AmgHierarchy(*s["A"], symmetric=False, solver="bicgstab", vcycle_prec=case["prec"])
    elif kind == "plain":
        s["H"] = AmgHierarchy(*s["A"], precondition=0)
    elif kind == "oneshot":
        s["kw"] = dict(vcycle_prec=case["prec"])
    else:
        s["H"] = AmgHierarchy(*s["A"], vcycle_prec=case["prec"])
    return s


def run(s):
    kind = s["kind"]
    if kind in ("solve", "plain"):
        return s["H"].solve(s["b"], s["tol"])[0]
    if kind in ("step", "systems"):
        s["H"].update_values(s["A"][2])
        return s["H"].solve(s["b"], s["tol"])[0]
    if kind == "oneshot":
        finalize()                       # the program meets this pattern for the first time
        return solve(s["A"], s["b"], s["tol"], **s["kw"])[0]
    if kind == "convection":
        x, _ = s["H"].solve(s["b"], s["tol"])
        lam, _ = s["H"].solve_adjoint(s["g"], s["tol"])
        return [x, lam, s["H"].pattern_grad(lam, x)]
    if kind == "vcycle":
        return s["H"].apply_vcycle(s["b"])
    theta = s["theta"].detach().requires_grad_(True)
    val = M.diffusion_values_torch(torch.exp(theta))
    x = amg_solve(s["A"][0], s["A"][1], val, s["b"], s["tol"], **s["kw"])
    loss = 0.5 * (x - s["target"]).square().sum()
    loss.backward()
    return [loss.detach(), x.detach(), theta.grad]


# ------------------------------------------------------- what a pass needs

def work(case):
    """Bytes and operations of one pass with every input read once, every
    output written once, and the products with A counted once per solve."""
    if case["kind"] == "plain":
        n = case["N"]
        nnz = 3 * n - 2
    else:
        N, d = case["N"], case["d"]
        n = N ** d
        nnz = (2 * d + 1) * n - 2 * d * N ** (d - 1)
    k = case.get("cols", 1)
    vals = nnz * (k if case["kind"] == "systems" else 1)
    solves = 2 if case["kind"] in ("train", "convection") else 1
    b = 4 * (nnz + n + 1) + 8 * vals + 16 * n * k * solves
    if case["kind"] == "convection":
        b += 8 * nnz
    if case["kind"] == "train":
        b += 16 * n
    return dict(bytes=b, flops=2 * nnz * k * solves)


# ------------------------------------------------ the answers in 64 bits

def _csr(A):
    n = len(A[0]) - 1
    return torch.sparse_csr_tensor(A[0], A[1], A[2].contiguous(), (n, n))


def _diagonal(A):
    rows = torch.repeat_interleave(torch.arange(len(A[0]) - 1, device=DEV), (A[0][1:] - A[0][:-1]).long())
    return A[2][A[1] == rows]


def _transposed(A):
    n = len(A[0]) - 1
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), (A[0][1:] - A[0][:-1]).long())
    order = torch.argsort(A[1].long() * n + rows)
    rp = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(A[1], minlength=n), dim=0)
    return rp, rows[order].to(torch.int32), A[2][order]


def _cg(A, b):
    """Diagonally scaled CG in 64 bits, restarted from its true residual until that stops falling."""
    S, w = _csr(A), 1.0 / _diagonal(A)
    w = w[:, None] if b.dim() == 2 else w
    x, best, kept = torch.zeros_like(b), math.inf, None
    for _ in range(4):
        r = b - S @ x
        now = float((r.norm(dim=0) / b.norm(dim=0)).max())
        if now >= 0.5 * best:
            break
        best, kept = now, x
        x = x.clone()
        z = w * r
        p, rz, r0 = z.clone(), (r * z).sum(dim=0), r.norm(dim=0)
        for it in range(20000):
            q = S @ p
            pq = (p * q).sum(dim=0)
            alpha = torch.where(pq > 0, rz / pq, torch.zeros_like(pq))
            x += alpha * p
            r -= alpha * q
            if it % 20 == 19 and bool((r.norm(dim=0) <= 1e-13 * r0).all()):
                break
            z = w * r
            new = (r * z).sum(dim=0)
            p = z + torch.where(rz > 0, new / rz, torch.zeros_like(rz)) * p
            rz = new
    return kept if kept is not None else x


def _bicgstab(A, b):
    """Diagonally scaled BiCGSTAB in 64 bits, restarted from its true residual until that stops falling."""
    S, w = _csr(A), 1.0 / _diagonal(A)
    x, best, kept = torch.zeros_like(b), math.inf, torch.zeros_like(b)
    for _ in range(8):
        r = b - S @ x
        now = float(r.norm() / b.norm())
        if not now < 0.5 * best:
            break
        best, kept = now, x
        x = x.clone()
        rh, p, rho, r0 = r.clone(), r.clone(), (r * r).sum(), r.norm()
        for it in range(4000):
            y = w * p
            v = S @ y
            alpha = rho / (rh * v).sum()
            s = r - alpha * v
            z = w * s
            t = S @ z
            omega = (t * s).sum() / (t * t).sum()
            x += alpha * y + omega * z
            r = s - omega * t
            if it % 20 == 19 and not bool(r.norm() > 1e-11 * r0):
                break
            new = (rh * r).sum()
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            rho = new
    return kept


def exact(case, seed):
    kind = case["kind"]
    if kind == "vcycle":
        return None  # no value apart from the hierarchy that the library chooses
    s = _inputs(case, seed)
    A, b = s["A"], s["b"]
    if kind == "systems":
        x = torch.empty_like(b)
        for c in range(case["cols"]):
            x[:, c] = _cg((A[0], A[1], A[2][:, c]), b[:, c].contiguous())
        return x
    if kind == "convection":
        x, lam = _bicgstab(A, b), _bicgstab(_transposed(A), s["g"])
        rows = torch.repeat_interleave(torch.arange(len(b), device=DEV), (A[0][1:] - A[0][:-1]).long())
        return [x, lam, -lam[rows] * x[A[1].long()]]
    if kind == "train":
        theta = s["theta"].detach().requires_grad_(True)
        val = _diffusion_values(torch.exp(theta), A[2])
        M64 = (A[0], A[1], val.detach())
        x = _cg(M64, b)
        lam = _cg(M64, x - s["target"])
        rows = torch.repeat_interleave(torch.arange(len(b), device=DEV), (A[0][1:] - A[0][:-1]).long())
        val.backward(-lam[rows] * x[A[1].long()])
        return [0.5 * (x - s["target"]).square().sum(), x, theta.grad]
    return _cg(A, b)
