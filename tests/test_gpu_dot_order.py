"""The sums of a MINRES iteration are grouped by the shape alone: whatever the tiles, and on its
own, in a group or in a persistent group launch, a solve leaves the same bits in its
workspace: vectors, scratch, bounds of the residual norm and scalar state."""
import pytest
import torch

import paper_2306_03574_amd.abac as abac

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
STEPS = 4
TOL = 1e-30


@pytest.fixture
def zeroed(monkeypatch):
    """Plans on cleared workspaces, with the default tiles."""
    empty = torch.empty

    def cleared(*a, **kw):
        return empty(*a, **kw).zero_() if kw.get("dtype") == torch.uint8 else empty(*a, **kw)

    monkeypatch.setenv("ABAC_TUNE", "0")
    monkeypatch.setattr(torch, "empty", cleared)


def _begun(nx, ny, nt, prec, batch, tiles=None):
    p = abac.Plan(nx, ny, nt, alpha=1e-2, prec=prec, batch=batch, device=DEV)
    if tiles:
        p.set_tiles(**tiles)
    f = abac.fill_normal(p.empty(), 17)
    p.begin(f, p.empty(), tol=TOL, maxit=100)
    return p


def _bits(p):
    """Every byte of the workspace up to the last right-hand side's scalar state: what lies behind
    are the partial sums themselves.  The state is found by its squared tolerance."""
    torch.cuda.synchronize()
    skip = -p.workspace.data_ptr() % 256
    words = p.workspace[skip:skip + (p.workspace.numel() - skip) // 8 * 8].view(torch.int64).clone()
    p.finish()
    tol2 = torch.tensor([TOL * TOL], dtype=torch.float64).view(torch.int64).item()
    at = (words == tol2).nonzero().flatten()
    assert at.numel() == p.batch
    return words[:int(at[-1]) + 1]


# x lengths 64 .. 4096: sequences of 8 to 256 threads, so units of eight row pairs to a row pair
# over four waves; (31, 15, 8): fewer row pairs than a wide tile takes
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,nt,batch", [(31, 15, 8, 2), (63, 31, 16, 1), (127, 7, 32, 1), (255, 15, 8, 2),
                                            (511, 7, 8, 1), (1023, 0, 32, 2), (2047, 0, 16, 1)])
def test_first_pass_tiles(zeroed, nx, ny, nt, batch, prec):
    first, ran = None, 0
    for wg in (64, 128, 256, 512, 1024):
        print(f"[case] dot order nx={nx} ny={ny} nt={nt} batch={batch} prec={prec} wg_x={wg}", flush=True)
        try:
            p = _begun(nx, ny, nt, prec, batch, {"dstx_fwd": wg})
        except abac.AbacError:
            continue   # not a legal tile
        p.advance(STEPS)
        bits = _bits(p)
        first = bits if first is None else first
        assert torch.equal(bits, first), wg
        ran += 1
    assert ran >= 2


# separate passes, fused passes with 128 and 512 threads, 1D
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_group_and_persistent(zeroed, prec):
    # (255, 63, 32) and (31, 31, 1024): more partials than a persistent block has threads
    shapes = [(127, 31, 16, 2), (255, 63, 32, 1), (31, 31, 1024, 1), (127 if prec == "fp32" else 63,) * 2 + (16, 1),
              (1023, 0, 16, 1)]
    solo = []
    for s in shapes:
        print(f"[case] solo {s} {prec}", flush=True)
        p = _begun(*s[:3], prec, s[3])
        p.advance(STEPS)
        solo.append(_bits(p))
    for how in ("advance", "run"):
        print(f"[case] group {how} {prec}", flush=True)
        plans = [_begun(*s[:3], prec, s[3]) for s in shapes]
        g = abac.Group(device=DEV)
        g.set(plans)
        getattr(g, how)(STEPS)
        torch.cuda.synchronize()
        if how == "run":
            assert not g.check()
        for s, p, bits in zip(shapes, plans, solo):
            assert torch.equal(_bits(p), bits), (how, s)
        g.close()
