"""Where a batch fills the GPU the matvec marches over several chunks of time levels per block and
still sums them one by one: batched solves equal single ones bit by bit."""
import pytest
import torch

from paper_2306_03574_amd.abac import Plan, fill_normal

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# marches of 2 and 4 chunks of 2 levels; at nt = 8 a march ends within its chunks
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,nt,batch", [(255, 15, 32, 32), (255, 15, 32, 64), (31, 31, 8, 128), (63, 7, 16, 300),
                                            (1023, 0, 16, 256)])
def test_batch_equals_solo(nx, ny, nt, batch, prec):
    print(f"[case] batch march nx={nx} ny={ny} nt={nt} batch={batch} prec={prec}", flush=True)
    p = Plan(nx, ny, nt, alpha=1e-2, prec=prec, batch=batch, device=DEV)
    one = Plan(nx, ny, nt, alpha=1e-2, prec=prec, device=DEV)
    f = fill_normal(p.empty(), 71)
    for run in (lambda q, g: q.solve(g, tol=1e-8, maxit=100), lambda q, g: q.gmres(g, tol=1e-6, maxit=30, restart=5)):
        u, iters, relres, status = run(p, f)
        for b in (0, batch // 2, batch - 1):
            v, i1, r1, s1 = run(one, f[b:b + 1].contiguous())
            torch.cuda.synchronize()
            assert (i1[0], r1[0], s1[0]) == (iters[b], relres[b], status[b])
            assert torch.equal(u[b], v[0])
