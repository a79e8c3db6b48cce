"""Characteristic reconstruction around a cell that is not a physical state (its
pressure negative or not a number): its own edges are not numbers, its neighbours' slopes vanish, and a PLM step agrees with the CPU oracle in
which entries hold NaN and, to relative L1 1e-12 per array, in all others.  With PPM a
NaN in the stencil reaches the edges, and the NaN entries agree."""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs

pytestmark = pytest.mark.gpu

CELL = (3 + 5, 3 + 6, 3 + 7)


@pytest.mark.parametrize("kind", ["negative pressure", "energy NaN", "energy -NaN"])
@pytest.mark.parametrize("recon,path", [("plm", "fused"), ("plm", "unfused"), ("ppm", "fused")])
def test_around_a_nonphysical_cell(orc, recon, path, kind):
    import torch

    from paper_2005_06651_amd import athmhd
    dev = torch.device("cuda:0")
    b = inputs.smooth_random(n=(20, 14, 11), seed=9, ng=3)
    kw = dict(integrator="rk1", recon=recon, riemann="roe")
    cfg = orc.cfg_for(b, charac=True, **kw)
    rc, rb = orc.prim2cons(orc.cfg_for(b, **kw), b.prim, b.bface), b.bface.copy()
    rc[(4,) + CELL] = {"negative pressure": 0.01, "energy NaN": np.nan, "energy -NaN": -np.nan}[kind]
    tc, tb = torch.from_numpy(rc.copy()).to(dev), torch.from_numpy(rb.copy()).to(dev)
    assert orc.step(cfg, rc, rb, 1e-3) > 0
    s = athmhd.Solver(b.n, b.ng, b.dx, b.gamma, charac=True, kernel_path=path, **kw)
    s.step(tc, tb, 1e-3)
    with pytest.raises(athmhd.NonPhysicalState):
        s.newdt(tc, tb)
    s.close()
    a = (slice(None),) + b.active
    for x, y in ((tc.cpu().numpy()[a], rc[a]), (tb.cpu().numpy()[a], rb[a])):
        bad = ~np.isfinite(y)
        assert np.array_equal(bad, ~np.isfinite(x)), (int(bad.sum()), int((~np.isfinite(x)).sum()))
        for v in range(len(x)):
            p, q = x[v][~bad[v]], y[v][~bad[v]]
            assert recon == "ppm" or float(np.abs(p - q).sum()) <= 1e-12 * float(np.abs(q).sum())
