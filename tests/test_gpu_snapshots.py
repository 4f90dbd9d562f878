"""Snapshots of a solve in host-mapped memory: a plan whose earlier solve is abandoned with
its iterations still queued must not take that solve's snapshots for the new one's, and a
ring of 16 snapshots must serve solves of any length."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# separate kernels, fused x-y passes, one workgroup per right-hand side
GRIDS = [(127, 0, 64), (31, 31, 32), (31, 0, 32)]


def _rhs(p, seed):
    src = np.stack([synth.random_source(p.nx, p.ny, p.nt, seed=seed + b)[0] for b in range(p.batch)])
    zero = torch.zeros((p.batch,) + p.level_shape, dtype=torch.float64, device=DEV)
    return p.build_rhs(torch.from_numpy(src).to(DEV), zero, zero)


@pytest.mark.parametrize("batch", [1, 3])
@pytest.mark.parametrize("nx,ny,nt", GRIDS)
def test_abandoned_solve(nx, ny, nt, batch):
    from paper_2306_03574_amd import Plan
    print(f"[case] abandoned solve nx={nx} ny={ny} nt={nt} batch={batch}", flush=True)
    p = Plan(nx, ny, nt, alpha=1e-2, batch=batch, device=DEV)
    f1, f2 = _rhs(p, 3), _rhs(p, 40)
    want, iters, relres, status = p.solve(f2, tol=1e-8, maxit=100)
    want = want.clone()
    u1, u2 = p.empty(), p.empty()
    p.begin(f1, u1, tol=1e-2, maxit=100)   # stops early: its snapshots say "done"
    p.advance(20)                          # more than the ring holds
    p.begin(f2, u2, tol=1e-8, maxit=100)   # at once, with those still queued
    steps = 0
    while not p.poll():
        p.advance(1)
        steps += 1
        assert steps < 200
        torch.cuda.synchronize()
    got = p.finish()
    assert got == (iters, relres, status)
    torch.cuda.synchronize()
    assert torch.equal(u2, want)
    assert steps <= max(iters) + 1


@pytest.mark.parametrize("nx,ny,nt", GRIDS)
def test_more_iterations_than_the_ring_holds(nx, ny, nt):
    """40 iterations of an unreachable tolerance, solved at once and enqueued ahead."""
    from paper_2306_03574_amd import Plan
    print(f"[case] long solve nx={nx} ny={ny} nt={nt}", flush=True)
    p = Plan(nx, ny, nt, alpha=1e-2, device=DEV)
    f = _rhs(p, 5)
    u1, it1, rr1, st1 = p.solve(f, tol=1e-30, maxit=40)
    u1 = u1.clone()
    u2 = p.empty()
    p.begin(f, u2, tol=1e-30, maxit=40)
    p.advance(40)
    it2, rr2, st2 = p.finish()
    torch.cuda.synchronize()
    assert it1 == it2 and rr1 == rr2 and st1 == st2
    assert torch.equal(u1, u2)


@pytest.mark.parametrize("nx,ny,nt", [(31, 15, 16), (15, 0, 16)])
def test_gmres_and_minres_take_turns(nx, ny, nt):
    """Both solvers post to the same ring: one plan that alternates them, with right-hand
    sides that stop apart (one is zero), gives what fresh plans give, also past the ring's
    length (40 GMRES steps in cycles of 3 post 54 snapshots)."""
    from paper_2306_03574_amd import Plan
    print(f"[case] alternating solvers nx={nx} ny={ny} nt={nt}", flush=True)

    def fresh():
        return Plan(nx, ny, nt, alpha=0.3, batch=3, device=DEV)

    def outcome(u, iters, relres, status):
        torch.cuda.synchronize()
        return u.clone(), iters, relres, status

    f = _rhs(fresh(), 9)
    f[1].zero_()
    calls = [lambda p: p.gmres(f, tol=1e-30, maxit=40, restart=3), lambda p: p.solve(f, tol=1e-8, maxit=200),
             lambda p: p.gmres(f, tol=1e-8, maxit=200)]
    want = [outcome(*c(fresh())) for c in calls]
    assert want[0][1] == [40, 0, 40] and want[0][3] == [-4, 0, -4] and want[2][3] == [0, 0, 0]
    p = fresh()
    for i in (0, 1, 2, 1, 0, 2):
        got = outcome(*calls[i](p))
        assert got[1:] == want[i][1:]
        assert torch.equal(got[0], want[i][0])


@pytest.mark.parametrize("restart", [1, 3])
def test_gmres_stops_in_the_last_column_of_a_cycle(restart):
    """maxit at the end of a cycle: the iterate of that column and ABAC_ENOCONV (-4), equal
    to what longer cycles give there."""
    from paper_2306_03574_amd import Plan
    p = Plan(31, 15, 16, alpha=0.3, device=DEV)
    f = _rhs(p, 9)
    u, iters, relres, status = p.gmres(f, tol=1e-30, maxit=restart, restart=restart)
    u = u.clone()
    assert iters == [restart] and status == [-4]
    v, iters2, relres2, status2 = p.gmres(f, tol=1e-30, maxit=restart, restart=15)
    torch.cuda.synchronize()
    assert (iters2, relres2, status2) == (iters, relres, status)
    assert torch.equal(u, v)


def test_tags_start_over():
    """The 16-bit tag of a plan's solves comes round again: a long solve that gets an earlier
    long solve's tag must wait for its own snapshots, of which the ring still holds the
    earlier one's last."""
    from paper_2306_03574_amd import Plan
    p = Plan(7, 7, 8, alpha=1e-2, device=DEV)
    f1, f2 = _rhs(p, 3), _rhs(p, 40)
    want = p.solve(f2, tol=1e-30, maxit=40)[1:]
    p = Plan(7, 7, 8, alpha=1e-2, device=DEV)
    u = p.empty()
    p.solve(f1, u, tol=1e-30, maxit=40)       # tag 1
    zero = torch.zeros_like(f1)
    for n in range(65535):                    # a zero right-hand side stops in the set-up
        p.solve(zero, u)
        if n % 16384 == 0:
            print(f"[progress] {n} solves", flush=True)
    got = p.solve(f2, u, tol=1e-30, maxit=40)[1:]
    assert got == want
