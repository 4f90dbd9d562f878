"""The timed cases of this framework: what its users have it do, through its public
entry points (Plan, Group), over the sizes it supports.

A case is a dict of plain values:
  kind     "solve":     right-hand side assembly, then MINRES to 1e-8 (Plan.build_rhs, Plan.solve)
           "gmres":     the same with GMRES and the block alpha-circulant preconditioner
           "operators": z = P^{-1} r and y = A z, one step of a caller's own Krylov method
           "group":     solves of several grids advanced together (Plan.begin, Group.advance)
  nx, ny, nt   interior grid points (ny = 0: 1D) and time levels
  alpha, prec, batch   as Plan takes them
  source   "noise": i.i.d. N(0, 1); "field": a smooth random field; "smoothed": N(0, 1)
           after three weighted-Jacobi sweeps per level; "standing": the standing wave
           sin(pi x) [sin(pi y)] sin(pi t) with N(0, 0.1^2) source noise
  coef     true: a variable coefficient that stays within some 10 % of its mean
  members  (group) the members' "nx x ny x nt @ alpha", separated by blanks
"""
import math

import numpy as np
import torch

from paper_2306_03574_amd.abac import Group, Plan

TOL, MAXIT = 1e-8, 500
DEV = "cuda:0"


def _case(kind, nx, ny, nt, prec="fp64", alpha=1e-3, batch=1, source="noise", coef=False, members=""):
    return {"kind": kind, "nx": nx, "ny": ny, "nt": nt, "prec": prec, "alpha": alpha, "batch": batch,
            "source": source, "coef": coef, "members": members}


def listed():
    return [
        # the smallest solve in use: one 1D problem, all latency
        dict(_case("solve", 63, 0, 64, source="standing"), name="1d_63x64"),
        # the same problem for many right-hand sides at once: throughput of tiny solves
        dict(_case("solve", 63, 0, 64, batch=256, source="standing"), name="1d_63x64_batch256"),
        # requests of a serving mix, FP32 transforms: a 1D and a small 2D grid, launch-bound
        dict(_case("solve", 1023, 0, 256, "fp32", 1e-2), name="1d_1023x256_fp32"),
        dict(_case("solve", 63, 63, 64, "fp32", 1e-2), name="2d_63x63x64_fp32"),
        # a ragged 2D grid: a long x axis, a short y axis
        dict(_case("solve", 127, 31, 256, source="field"), name="2d_127x31x256"),
        # the variable-coefficient equation: more iterations than the resident basis holds
        dict(_case("solve", 63, 63, 64, source="field", coef=True), name="2d_63x63x64_coef"),
        # seven grids of the serving mix solved as one group
        dict(_case("group", 0, 0, 0, "fp32", members="63x63x256@1e-2 127x127x64@1e-3 255x0x512@1e-3 1023x0x256@1e-2 "
                   "63x63x64@1e-3 255x0x256@1e-2 127x127x256@1e-3"), name="group7_fp32"),
        # the operators on their own, for a caller's own Krylov method
        dict(_case("operators", 255, 255, 256), name="operators_255x255x256"),
        # the non-symmetric solver that the symmetric one is compared with
        dict(_case("gmres", 255, 127, 128, source="field"), name="gmres_255x127x128"),
        # the medium solve, FP64 throughout
        dict(_case("solve", 255, 255, 256), name="2d_255x255x256"),
        # 64 right-hand sides of one grid
        dict(_case("solve", 127, 127, 128, batch=64, source="smoothed"), name="2d_127x127x128_batch64"),
        # the large solve, FP32 transforms and FP64 Krylov vectors
        dict(_case("solve", 511, 511, 512, "fp32", source="field"), name="2d_511x511x512_fp32"),
    ]


def _unknowns(c):
    if c["kind"] == "group":
        return sum(nt * nx * max(ny, 1) for nx, ny, nt, _ in _members(c))
    return c["batch"] * c["nt"] * c["nx"] * max(c["ny"], 1)


def draw(rng):
    """One more case of the same ranges; its unknowns are spread over their logarithm,
    up to a quarter of the largest listed case's."""
    kind = rng.choice(["solve"] * 5 + ["coef", "operators", "gmres", "group"])
    while True:
        alpha = rng.choice([1e-2, 1e-3])
        prec = rng.choice(["fp64", "fp32"])
        source = rng.choice(["noise", "field"])
        nt = 2 ** rng.randint(3, 10)
        oned = rng.random() < 0.35
        if kind == "group":
            shapes = []
            for _ in range(rng.randint(2, 12)):
                if rng.random() < 0.5:
                    nx, ny = 2 ** rng.randint(7, 10) - 1, 0
                else:
                    nx = 2 ** rng.randint(5, 7) - 1
                    ny = rng.choice([nx, 2 ** rng.randint(4, 7) - 1])
                shapes.append("%dx%dx%d@%s" % (nx, ny, 2 ** rng.randint(6, 9), rng.choice(["1e-2", "1e-3"])))
            c = _case("group", 0, 0, 0, prec, members=" ".join(shapes))
        elif kind == "coef":
            nx = 2 ** rng.randint(4, 7) - 1
            ny = 0 if oned else 2 ** rng.randint(4, 6) - 1
            c = _case("solve", nx, ny, 2 ** rng.randint(5, 8), "fp64", 1e-3, rng.choice([1, 1, 2, 4]), "field", True)
        else:
            nx = 2 ** rng.randint(3, 12) - 1 if oned else 2 ** rng.randint(3, 9) - 1
            ny = 0 if oned else rng.choice([nx, 2 ** rng.randint(3, 9) - 1])
            batch = rng.choice([1, 1, 1, 2, 3, 8, 31, 64, 200])
            if kind in ("operators", "gmres"):
                prec = "fp64"
            if kind == "gmres":
                batch = min(batch, 8)
            c = _case(kind, nx, ny, nt, prec, alpha, batch, source)
        if 3000 <= _unknowns(c) <= 2 ** 25 and rng.random() < 0.25 + 0.75 * math.log(_unknowns(c)) / math.log(2 ** 25):
            return c


def _members(case):
    out = []
    for m in case["members"].split():
        grid, alpha = m.split("@")
        nx, ny, nt = (int(v) for v in grid.split("x"))
        out.append((nx, ny, nt, float(alpha)))
    return out


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _points(n):
    return torch.arange(1, n + 1, dtype=torch.float64, device=DEV) / (n + 1)


def _source(kind, nx, ny, nt, batch, seed):
    """Source samples [batch][nt][ny][nx] and the two initial levels."""
    gen = torch.Generator(DEV)
    gen.manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(shape, dtype=torch.float64, device=DEV, generator=gen)

    level = (ny, nx) if ny else (nx,)
    psi0 = torch.zeros((batch,) + level, dtype=torch.float64, device=DEV)
    psi1 = torch.zeros_like(psi0)
    if kind == "field":
        # a field of correlation length 0.1 from its leading sine (space) and cosine
        # (time) modes, unit RMS
        k = 12
        damp = torch.exp(-0.0493 * torch.arange(1, k + 1, dtype=torch.float64, device=DEV) ** 2)
        modes = torch.arange(1, k + 1, dtype=torch.float64, device=DEV)
        sx = torch.sin(math.pi * modes[:, None] * _points(nx)) * damp[:, None]
        ct = torch.cos(math.pi * (modes[:, None] - 1) * torch.arange(nt, dtype=torch.float64, device=DEV) / nt) * damp[:, None]
        src = torch.empty((batch, nt) + level, dtype=torch.float64, device=DEV)
        for b in range(batch):
            if ny:
                sy = torch.sin(math.pi * modes[:, None] * _points(ny)) * damp[:, None]
                a = torch.matmul(ct.t().contiguous(), normal(k, k * k)).reshape(nt, k, k)     # [t][q][p]
                a = torch.matmul(a.reshape(nt * k, k), sx).reshape(nt, k, nx)                  # [t][q][x]
                a = torch.matmul(sy.t().contiguous(), a.permute(1, 0, 2).reshape(k, nt * nx))  # [y][t x]
                src[b] = a.reshape(ny, nt, nx).permute(1, 0, 2)
            else:
                src[b] = torch.matmul(torch.matmul(ct.t().contiguous(), normal(k, k)), sx)
            src[b] /= src[b].square().mean().sqrt()
        return src, psi0, psi1
    src = normal(batch, nt, *level)
    if kind == "standing":
        src *= 0.1
        s = torch.sin(math.pi * _points(nx))
        if ny:
            s = torch.sin(math.pi * _points(ny))[:, None] * s
            t = torch.arange(nt, dtype=torch.float64, device=DEV) / nt
            src += math.pi ** 2 * torch.sin(math.pi * t)[:, None, None] * s
        psi1 += math.pi * s
    elif kind == "smoothed":
        for _ in range(3):
            p = torch.nn.functional.pad(src, (1, 1, 1, 1))
            nb = p[..., :-2, 1:-1] + p[..., 2:, 1:-1] + p[..., 1:-1, :-2] + p[..., 1:-1, 2:]
            src = src / 3.0 + nb / 6.0
    return src, psi0, psi1


def _coefficient(nx, ny, seed):
    """Face values of a smooth coefficient a > 0 and its mean over the grid points."""
    c = np.random.default_rng(int(seed)).uniform(0.5, 1.0, size=3)
    x, xh = np.arange(1, nx + 1) / (nx + 1), (np.arange(nx + 1) + 0.5) / (nx + 1)
    if not ny:
        def a(x):
            return 2.0 * (1.0 + 0.1 * (c[0] * np.sin(3 * x) ** 2 + c[1] * x))
        return a(xh)[None], None, float(a(x).mean())

    def a(x, y):
        return 2.0 * (1.0 + 0.1 * (c[0] * np.sin(3 * x) ** 2 + c[1] * y * y - c[2] * x * y))
    y, yh = np.arange(1, ny + 1) / (ny + 1), (np.arange(ny + 1) + 0.5) / (ny + 1)
    return a(xh[None, :], y[:, None]), a(x[None, :], yh[:, None]), float(a(x[None, :], y[:, None]).mean())


def prepare(case, seed):
    c = case
    if c["kind"] == "group":
        group = Group(device=DEV)
        plans = [Plan(nx, ny, nt, alpha=al, prec=c["prec"], device=DEV) for nx, ny, nt, al in _members(c)]
        srcs = [_source(c["source"], p.nx, p.ny, p.nt, 1, 1000 * seed + i) for i, p in enumerate(plans)]
        return {"case": c, "group": group, "plans": plans, "sources": srcs, "f": [p.empty() for p in plans],
                "u": [p.empty() for p in plans]}
    plan = Plan(c["nx"], c["ny"], c["nt"], alpha=c["alpha"], prec=c["prec"], batch=c["batch"], device=DEV)
    if c["coef"]:
        plan.set_coefficient(*_coefficient(c["nx"], c["ny"], seed))
    src, psi0, psi1 = _source(c["source"], c["nx"], c["ny"], c["nt"], c["batch"], seed)
    return {"case": c, "plan": plan, "src": src, "psi0": psi0, "psi1": psi1, "f": plan.empty(), "u": plan.empty()}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    s, kind = state, state["case"]["kind"]
    if kind == "group":
        group, plans = s["group"], s["plans"]
        for p, src, f, u in zip(plans, s["sources"], s["f"], s["u"]):
            p.build_rhs(*src, f=f)
            p.begin(f, u, tol=TOL, maxit=MAXIT)
        group.set(plans)
        done = False
        while not done:
            group.advance(4)
            torch.cuda.current_stream().synchronize()
            done = all([p.poll() for p in plans])
        return {"u": s["u"], "iterations": torch.tensor([p.finish()[0][0] for p in plans])}
    plan = s["plan"]
    if kind == "operators":
        z = plan.apply_Pinv(s["src"], s["f"])
        return {"z": z, "y": plan.apply_A(z, s["u"])}
    f = plan.build_rhs(s["src"], s["psi0"], s["psi1"], f=s["f"])
    solver = plan.gmres if kind == "gmres" else plan.solve
    u, iters, _, _ = solver(f, s["u"], tol=TOL, maxit=MAXIT)
    return {"u": u, "iterations": torch.tensor(iters)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _apply_flops(nx, ny, nt, prec_applies, matvecs):
    """Per right-hand side: a P^{-1} is two sine transforms along each space axis, four
    real FFTs over time and two complex scalings per value; a matvec is one stencil."""
    n = nt * nx * max(ny, 1)
    space = 2 * 2.5 * (math.log2(2 * (nx + 1)) + (math.log2(2 * (ny + 1)) if ny else 0))
    return n * (prec_applies * (space + 4 * 2.5 * math.log2(nt) + 16) + matvecs * (16 if ny else 10))


def work(case):
    """Inputs read once and outputs written once, and the operators' arithmetic; a solve
    is counted with eight iterations, what these problems take (6 to 10)."""
    c = case
    if c["kind"] == "operators":
        return {"bytes": 3 * 8 * _unknowns(c), "flops": c["batch"] * _apply_flops(c["nx"], c["ny"], c["nt"], 1, 1)}
    grids = [m[:3] for m in _members(c)] if c["kind"] == "group" else [(c["nx"], c["ny"], c["nt"])] * c["batch"]
    return {"bytes": 2 * 8 * _unknowns(c), "flops": sum(_apply_flops(*g, 9, 8) for g in grids)}


# ---------------------------------------------------------------------------
# the same results in 64 bits, by other means
# ---------------------------------------------------------------------------

def _dst_matrix(n):
    k = torch.arange(1, n + 1, dtype=torch.float64, device=DEV)
    # the product of the indices is reduced mod 2(n+1) before it meets pi
    return torch.sin(math.pi * torch.remainder(k[:, None] * k, 2 * (n + 1)) / (n + 1)) * math.sqrt(2.0 / (n + 1))


def _dst(v, nx, ny):
    """Orthonormal sine transform along the space axes of [nt][ny][nx] (or [nt][nx])."""
    v = torch.matmul(v, _dst_matrix(nx))
    if ny:
        v = torch.matmul(v.transpose(-1, -2).contiguous(), _dst_matrix(ny)).transpose(-1, -2).contiguous()
    return v


def _kappa(nx, ny):
    """Eigenvalues of -Laplace_h in the sine basis."""
    kx = 4.0 * (nx + 1) ** 2 * torch.sin(0.5 * math.pi * _points(nx)) ** 2
    if not ny:
        return kx
    return 4.0 * (ny + 1) ** 2 * torch.sin(0.5 * math.pi * _points(ny))[:, None] ** 2 + kx


def _march(f, solve_L, apply_L):
    """T u = f level by level: L u_k = f_k + 2 u_{k-1} - L u_{k-2}."""
    u = torch.empty_like(f)
    for k in range(f.shape[0]):
        r = f[k].clone()
        if k >= 1:
            r += 2.0 * u[k - 1]
        if k >= 2:
            r -= apply_L(u[k - 2])
        u[k] = solve_L(r)
    return u


def _rhs(src, psi0, psi1, apply_L):
    tau = 1.0 / src.shape[0]
    f = tau * tau * src
    f[0] = 0.5 * tau * tau * src[0] + tau * psi1 + psi0
    f[1] -= apply_L(psi0)
    return f


def _solve_exact(nx, ny, nt, src, psi0, psi1):
    lam = 1.0 + 0.5 / nt ** 2 * _kappa(nx, ny)
    f = _rhs(_dst(src, nx, ny), _dst(psi0, nx, ny), _dst(psi1, nx, ny), lambda v: lam * v)
    return _dst(_march(f, lambda r: r / lam, lambda v: lam * v), nx, ny)


def _solve_exact_coef(nx, ny, nt, src, psi0, psi1, seed):
    axh, ayh, _ = _coefficient(nx, ny, seed)
    ny1, hx, hy = max(ny, 1), 1.0 / (nx + 1), 1.0 / (ny + 1)
    idx = np.arange(ny1 * nx).reshape(ny1, nx)
    L = np.eye(ny1 * nx)
    w = 0.5 / nt ** 2 * axh / hx ** 2
    L[idx, idx] += w[:, :-1] + w[:, 1:]
    L[idx[:, :-1], idx[:, 1:]] -= w[:, 1:-1]
    L[idx[:, 1:], idx[:, :-1]] -= w[:, 1:-1]
    if ny:
        w = 0.5 / nt ** 2 * ayh / hy ** 2
        L[idx, idx] += w[:-1] + w[1:]
        L[idx[:-1], idx[1:]] -= w[1:-1]
        L[idx[1:], idx[:-1]] -= w[1:-1]
    L = torch.from_numpy(L)
    chol = torch.linalg.cholesky(L)
    src, psi0, psi1 = (v.cpu().reshape(-1, ny1 * nx) for v in (src, psi0, psi1))
    f = _rhs(src, psi0[0], psi1[0], lambda v: L @ v)
    u = _march(f, lambda r: torch.cholesky_solve(r[:, None], chol)[:, 0], lambda v: L @ v)
    return u.reshape((nt, ny, nx) if ny else (nt, nx)).to(DEV)


def _pinv_exact(nx, ny, nt, alpha, r):
    """C^{-1/2} (C^{-1/2})^T r with complex FFTs over time."""
    t = torch.arange(nt, dtype=torch.float64, device=DEV)
    shape = (nt,) + (1,) * (2 if ny else 1)
    a = alpha ** (1.0 / nt)
    d = (a ** t).reshape(shape)
    w = torch.exp(torch.complex(torch.zeros_like(t), -2.0 * math.pi * t / nt)).reshape(shape)
    lam = 1.0 + 0.5 / nt ** 2 * _kappa(nx, ny)
    m = 1.0 / torch.sqrt(lam * (1.0 + a * a * w * w) - 2.0 * a * w)
    v = torch.fft.ifft(_dst(r, nx, ny) / d, dim=0) * m
    v = torch.fft.fft(v, dim=0).real * d * d
    v = torch.fft.ifft(torch.fft.fft(v, dim=0) * m, dim=0).real / d
    return _dst(v, nx, ny)


def _matvec_exact(nx, ny, nt, z):
    """Y T z, Y the time reversal."""
    h = [1.0 / (nx + 1)] + ([1.0 / (ny + 1)] if ny else [])
    lz = z.clone()
    for axis, hh in enumerate(h):
        dim, w = -1 - axis, 0.5 / nt ** 2 / hh ** 2
        n = z.shape[dim]
        lz += 2.0 * w * z
        lz.narrow(dim, 1, n - 1).sub_(w * z.narrow(dim, 0, n - 1))
        lz.narrow(dim, 0, n - 1).sub_(w * z.narrow(dim, 1, n - 1))
    y = lz.clone()
    y[1:] -= 2.0 * z[:-1]
    y[2:] += lz[:-2]
    return y.flip(0)


def exact(case, seed):
    """Solves: the solution of T u = f by marching it in time, in the sine basis or (variable
    coefficient) with a dense factorisation; the iteration counts have no such value."""
    c = case
    if c["kind"] == "group":
        us = [_solve_exact(nx, ny, nt, *(v[0] for v in _source(c["source"], nx, ny, nt, 1, 1000 * seed + i)))[None]
              for i, (nx, ny, nt, _) in enumerate(_members(c))]
        return {"u": us, "iterations": None}
    nx, ny, nt = c["nx"], c["ny"], c["nt"]
    src, psi0, psi1 = _source(c["source"], nx, ny, nt, c["batch"], seed)
    if c["kind"] == "operators":
        z = torch.stack([_pinv_exact(nx, ny, nt, c["alpha"], src[b]) for b in range(c["batch"])])
        return {"z": z, "y": torch.stack([_matvec_exact(nx, ny, nt, z[b]) for b in range(c["batch"])])}
    out = torch.empty_like(src)
    for b in range(c["batch"]):
        if c["coef"]:
            out[b] = _solve_exact_coef(nx, ny, nt, src[b], psi0[b], psi1[b], seed)
        else:
            out[b] = _solve_exact(nx, ny, nt, src[b], psi0[b], psi1[b])
    return {"u": out, "iterations": None}
