"""PPM stages of launches with no more workgroups than compute units run a
variant whose limiters have no branches.  A block alone takes it; the same
block many times over in one launch does not.  Both do the same operations, so
they may differ by the contraction of multiplies and adds only: bars of the
parity tests (relative L1 1e-12 per array, element by element 1e-10)."""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs

pytestmark = pytest.mark.gpu

MANY = 300  # blocks: more than the 256 compute units whatever a block's size


def _jumpy(n):
    """Density and pressure jumps over a smooth field, extrema in every line."""
    b = inputs.smooth_random(n=n, seed=sum(n) + 1, ng=3)
    rng = np.random.default_rng(3)
    jump = rng.integers(0, 2, size=b.prim[0].shape)
    b.prim[0] *= 1.0 + 3.0 * jump
    b.prim[4] *= 1.0 + 7.0 * (1 - jump)
    return b


@pytest.mark.parametrize("floors", [False, True])
@pytest.mark.parametrize("riemann", ["hlld", "hlle", "roe"])
@pytest.mark.parametrize("n", [(16, 12, 8), (17, 13, 5), (33, 25, 7), (5, 30, 3)])
def test_alone_equals_many(n, riemann, floors):
    import torch

    from paper_2005_06651_amd import athmhd
    # the jumps need the floors: without them Roe (and HLLD) leave the physical states
    b = _jumpy(n) if floors else inputs.smooth_random(n=n, seed=sum(n) + 1, ng=3)
    kw = dict(integrator="rk3", recon="ppm", riemann=riemann)
    dev = torch.device("cuda:0")
    out = []
    for nb in (1, MANY):
        s = athmhd.Solver(b.n, b.ng, b.dx, b.gamma, nblocks=nb, **kw)
        if floors:
            s.set_floors(1.5 * float(b.prim[0].min()), 1.5 * float(b.prim[4].min()))
        rep = (lambda x: torch.from_numpy(x).to(dev)) if nb == 1 else \
            (lambda x: torch.from_numpy(x).to(dev).expand(nb, *x.shape).contiguous())
        prim, face = rep(b.prim), rep(b.bface)
        s.fill_ghosts(prim, face)
        cons = s.prim2cons(prim, face)
        one = cons if nb == 1 else cons[0].contiguous()
        if nb == 1:
            dt = 0.3 * s.newdt(one, face)
        for _ in range(2):
            s.step(cons, face, dt)
        out.append((cons.cpu().numpy(), face.cpu().numpy()))
        s.close()
    a = b.active
    (c1, f1), (cn, fn) = out
    assert np.isfinite(c1).all()
    scale = np.mean([np.abs(f1[d][a]).mean() for d in range(3)])
    for one, many, floor in ((c1, cn, 0.0), (f1, fn, scale)):
        for q in (0, MANY // 2, MANY - 1):
            for x, y in zip(one, many[q]):
                x, y = x[a], y[a]
                mean = max(np.abs(y).mean(), floor)
                assert np.abs(x - y).mean() <= 1e-12 * mean
                assert np.max(np.abs(x - y) / (np.abs(y) + mean)) <= 1e-10
