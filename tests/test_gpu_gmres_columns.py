"""The longest GMRES cycle: the scalar steps sum one product per wave, and the fifteenth
column of a cycle fills all sixteen."""
import numpy as np
import pytest
import torch

from oracle.discretization import Grid
from oracle import allatonce as aao
from oracle import preconditioner as pc
from oracle import gmres as gm
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [14, 15, 16])
def test_iterates_around_a_full_cycle(k):
    """Bounds of the shorter cycles' test: 1e-10 for the iterate, 1e-9 for the residual (of
    5e-4, so four digits above the rounding of the products summed)."""
    from paper_2306_03574_amd import Plan
    nx, ny, nt, alpha = 15, 7, 16, 0.6
    g = Grid(nx, ny, nt)
    f = aao.build_rhs(g, *synth.random_source(nx, ny, nt, seed=23))
    ref = gm.gmres(lambda u: aao.apply_T(g, u), lambda y: pc.apply_C_inv(g, alpha, y), f, fixed_iters=k, restart=15)
    p = Plan(nx, ny, nt, alpha=alpha, device="cuda:0")
    u, iters, relres, status = p.gmres(torch.from_numpy(f[None]).to("cuda:0"), tol=1e-30, maxit=k, restart=15)
    torch.cuda.synchronize()
    got = u.cpu().numpy()[0]
    assert iters == [k] and status == [-4]
    assert np.max(np.abs(got - ref.x)) <= 1e-10 * np.max(np.abs(ref.x))
    assert abs(relres[0] - ref.relres) <= 1e-9 * ref.relres
