"""Slow convergence (several cycles of the resident basis, the tracked residual vector) where the
iterations are queued ahead, in a group and in persistent launches: count, residual and iterate
are bitwise those of Plan.solve."""
import numpy as np
import pytest
import torch

from test_gpu_slow_convergence import _problem

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MAXIT = 400
# separate 1D kernels, separate 2D kernels, fused x-y passes
GRIDS = [(127, 0, 64), (15, 7, 32), (31, 31, 16)]


def _plan(nx, ny, nt, alpha, prec):
    """A plan for two right-hand sides that stop apart, and those."""
    from paper_2306_03574_amd import Plan
    _, _, axh, ayh, abar, f = _problem(nx, ny, nt, 5.0, seed=9)
    _, _, _, _, _, f2 = _problem(nx, ny, nt, 5.0, seed=31)
    p = Plan(nx, ny, nt, alpha=alpha, prec=prec, batch=2, device=DEV)
    p.set_coefficient(axh, ayh, abar)
    return p, torch.from_numpy(np.stack([f, f2])).to(DEV)


def _drive(step, plans):
    for _ in range(MAXIT):
        step()
        torch.cuda.synchronize()
        if all(p.poll() for p in plans):
            return
    raise AssertionError("did not stop")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("alpha", [1e-3, 1e-1])
@pytest.mark.parametrize("tol", [2e-1, 1e-1, 3e-2])
def test_queued_and_grouped(tol, alpha, prec):
    from paper_2306_03574_amd import Group
    ref = []
    for g in GRIDS:
        print(f"[case] slow {g} tol={tol} alpha={alpha} {prec}: solve, queued", flush=True)
        p, f = _plan(*g, alpha, prec)
        u, *res = p.solve(f, tol=tol, maxit=MAXIT)
        torch.cuda.synchronize()
        assert res[2] == [0, 0]
        ref.append((u, *res))
        for ahead in (1, 7):
            v = p.empty()
            p.begin(f, v, tol=tol, maxit=MAXIT)
            _drive(lambda: p.advance(ahead), [p])
            assert list(p.finish()) == res
            assert torch.equal(u, v)
    assert max(max(r[1]) for r in ref) > 12   # beyond the first cycle
    for how, chunk in (("advance", 1), ("advance", 5), ("run", 1), ("run", 13)):
        print(f"[case] slow group {how} {chunk} tol={tol} alpha={alpha} {prec}", flush=True)
        members = [_plan(*g, alpha, prec) for g in GRIDS]
        us = [p.empty() for p, _ in members]
        for (p, f), u in zip(members, us):
            p.begin(f, u, tol=tol, maxit=MAXIT)
        group = Group(device=DEV)
        group.set([p for p, _ in members])
        _drive(lambda: getattr(group, how)(chunk), [p for p, _ in members])
        assert how == "advance" or not group.check()
        for (p, _), u, (u0, *res) in zip(members, us, ref):
            assert list(p.finish()) == res
            assert torch.equal(u, u0)
        group.close()
