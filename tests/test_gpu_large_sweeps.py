"""Sweeps whose blocks take more than one turn: forming the iterate in chunks of 4096
elements and the set-up's reversed copy, past 1024 blocks per right-hand side."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("nx,ny,nt", [(255, 127, 256), (511, 31, 512)])
def test_every_element_is_formed(nx, ny, nt):
    """relres is of the formed u, over the norm that the set-up sums.  Both are formed again
    from T u here, equal but for the rounding of T u: ||T|| is a few units and ||u|| is of the
    order of nt^2 ||f||."""
    from paper_2306_03574_amd import Plan
    print(f"[case] large sweeps nx={nx} ny={ny} nt={nt}", flush=True)
    p = Plan(nx, ny, nt, alpha=1e-3, device=DEV)
    src = synth.random_source(p.nx, p.ny, p.nt, seed=7)[0]
    zero = torch.zeros((1,) + p.level_shape, dtype=torch.float64, device=DEV)
    f = p.build_rhs(torch.from_numpy(src[None]).to(DEV), zero, zero)
    u = torch.full_like(f, float("nan"))
    u, iters, relres, status = p.solve(f, u, tol=1e-8, maxit=60)
    r = f - p.apply_T(u)
    torch.cuda.synchronize()
    assert status == [0] and relres[0] <= 1e-8
    assert abs(float(r.norm() / f.norm()) - relres[0]) <= 100 * np.finfo(float).eps * nt ** 2
