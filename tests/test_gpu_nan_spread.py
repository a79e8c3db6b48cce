"""A cell that is not a number makes every face state formed from it one,
whatever its sign bit: after a PPM step the same cells and faces hold NaN as in the
CPU oracle, in the general stage kernel (a block many times over) and in the
variant of a launch with a compute unit per workgroup (the block alone)."""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nblocks", [1, 300])
@pytest.mark.parametrize("var", [0, 2, 4])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_nan_reaches_what_the_stencil_reaches(orc, sign, var, nblocks):
    import torch

    from paper_2005_06651_amd import athmhd
    b = inputs.smooth_random(n=(24, 20, 16), seed=5, ng=3)
    kw = dict(integrator="rk1", recon="ppm", riemann="roe")
    cfg = orc.cfg_for(b, **kw)
    cons, face = orc.prim2cons(cfg, b.prim, b.bface), b.bface.copy()
    dt, _ = orc.newdt(cfg, cons, face)
    cons[var, 3 + 8, 3 + 10, 3 + 12] = np.copysign(np.nan, sign)
    dev = torch.device("cuda:0")
    tc, tb = (torch.from_numpy(x).to(dev).expand(nblocks, *x.shape).contiguous() for x in (cons, face))
    assert orc.step(cfg, cons, face, dt) > 0
    s = athmhd.Solver(b.n, b.ng, b.dx, b.gamma, nblocks=nblocks, **kw)
    s.step(tc, tb, dt)
    a = (slice(None),) + b.active
    got = [np.isnan(x[nblocks - 1].cpu().numpy()[a]) for x in (tc, tb)]
    want = [np.isnan(x[a]) for x in (cons, face)]
    assert want[0].any()
    for x, y in zip(got, want):
        assert np.array_equal(x, y), (int(x.sum()), int(y.sum()))
    s.close()
