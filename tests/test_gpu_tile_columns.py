"""The 34 x 15 thread tile (32 x 13 active columns) one column more, one less and
as many, with a ragged last x3 segment, against the CPU oracle.  A small block
alone runs on the smaller tile; these block counts fill the chip once with
the larger one and more than once with the smaller, so that the plan takes the
larger for every reconstruction.

Bar: relative L1 1e-12 per array, element by element 1e-10 (the bars of the other
parity tests)."""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("integ,recon,riemann", [("vl2", "plm", "hlld"), ("rk3", "ppm", "hlle"), ("rk2", "dc", "hlld")])
@pytest.mark.parametrize("n,nb", [((31, 13, 9), 85), ((32, 13, 9), 85), ((33, 13, 9), 42), ((32, 25, 7), 64),
                                  ((32, 26, 7), 64), ((33, 25, 7), 32)])
def test_larger_tile_matches_oracle(orc, monkeypatch, n, nb, integ, recon, riemann):
    import torch

    from paper_2005_06651_amd import athmhd
    monkeypatch.setenv("ATHMHD_KZ", "4")
    b = inputs.smooth_random(n=n, seed=sum(n), ng=3)
    kw = dict(integrator=integ, recon=recon, riemann=riemann)
    cfg = orc.cfg_for(b, **kw)
    cons = orc.prim2cons(cfg, b.prim, b.bface)
    dev = torch.device("cuda:0")
    tc, tb = (torch.from_numpy(x).to(dev).expand(nb, *x.shape).contiguous() for x in (cons, b.bface))
    s = athmhd.Solver(b.n, b.ng, b.dx, b.gamma, nblocks=nb, **kw)
    rc, rb = cons.copy(), b.bface.copy()
    for _ in range(2):
        dt, _ = orc.newdt(cfg, rc, rb)
        assert orc.step(cfg, rc, rb, dt) == 0
        s.step(tc, tb, dt)
    a = b.active
    act = (slice(None), slice(None)) + a
    assert torch.equal(tc[act], tc[:1][act].expand(nb, -1, -1, -1, -1))
    assert torch.equal(tb[act], tb[:1][act].expand(nb, -1, -1, -1, -1))
    scale = np.mean([np.abs(rb[c][a]).mean() for c in range(3)])
    for got, ref, floor in ((tc[nb - 1].cpu().numpy(), rc, 0.0), (tb[nb - 1].cpu().numpy(), rb, scale)):
        for x, y in zip(got, ref):
            x, y = x[a], y[a]
            mean = max(np.abs(y).mean(), floor)
            assert np.abs(x - y).mean() <= 1e-12 * mean
            assert np.max(np.abs(x - y) / (np.abs(y) + mean)) <= 1e-10
    s.close()
