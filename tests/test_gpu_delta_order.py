"""delta_j is summed in the first transform pass where the vectors are small, by a scalar step
where they are not: in the same order, so a batch equals its right-hand sides bit by bit
also where only the batch is too large for the former."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,nt,batch", [(63, 31, 64, 40), (63, 63, 1024, 2), (1023, 0, 256, 20), (127, 127, 128, 3)])
def test_batch_equals_solo_across_the_limit(nx, ny, nt, batch, prec):
    from paper_2306_03574_amd import Plan
    unknowns = nx * max(ny, 1) * nt
    assert unknowns * 8 <= 32 << 20 < unknowns * 8 * batch
    print(f"[case] delta order nx={nx} ny={ny} nt={nt} batch={batch} prec={prec}", flush=True)
    p = Plan(nx, ny, nt, alpha=1e-2, prec=prec, batch=batch, device=DEV)
    one = Plan(nx, ny, nt, alpha=1e-2, prec=prec, device=DEV)
    src = np.stack([synth.random_source(nx, ny, nt, seed=60 + b)[0] for b in range(batch)])
    zero = torch.zeros((batch,) + p.level_shape, dtype=torch.float64, device=DEV)
    f = p.build_rhs(torch.from_numpy(src).to(DEV), zero, zero)
    u, iters, relres, status = p.solve(f, tol=1e-8, maxit=100)
    for b in (0, batch - 1):
        v, i1, r1, s1 = one.solve(f[b:b + 1].contiguous(), tol=1e-8, maxit=100)
        torch.cuda.synchronize()
        assert (i1[0], r1[0], s1[0]) == (iters[b], relres[b], status[b])
        assert torch.equal(u[b], v[0])
