"""Reverse mode on lines short enough for a workgroup to hold them whole (up to
64 faces along x1, 32 with PLM and 16 with donor cell along x2 and x3), at the
lengths where that form and the lines laid end to end take turns, and on blocks
with few cells along x1, whose lines are numbered across x1 and the other direction.

Oracle: the transposition identity with the CPU oracle's directional
derivatives, as in the layout test (1e-12 of the sum of magnitudes); and a block of
copies of a short one, whose lines are laid end to end, gives the same cotangents to
1e-13 of their largest."""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs
from test_gpu_adjoint import active_masks, athmhd, gpu_vjp, oracle_jvp, random_active, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu

SCHEMES = [("vl2", "plm", "hlld"), ("rk1", "plm", "hlle"), ("rk1", "dc", "hlld")]


@pytest.mark.parametrize("n", [(1, 2, 1), (1, 40, 21), (2, 37, 5), (3, 1, 130), (64, 1, 2), (65, 32, 1), (62, 33, 16),
                               (31, 10, 17), (21, 11, 32), (9, 16, 31)])
@pytest.mark.parametrize("integ,recon,rs", SCHEMES)
def test_transposition_over_short_lines(torch_dev, athmhd, orc, n, integ, recon, rs):  # noqa: F811
    torch, dev = torch_dev
    blk = inputs.smooth_random(n=n, seed=23, ng=2)
    kw = dict(integrator=integ, recon=recon, riemann=rs, ct_eps=1e-3)
    cfg = orc.cfg_for(blk, **kw)
    cons = orc.prim2cons(cfg, blk.prim, blk.bface)
    dt = orc.newdt(cfg, cons, blk.bface)[0]
    mc, mb = active_masks(blk.n, blk.ng)
    s = athmhd.Solver(blk.n, blk.ng, blk.dx, blk.gamma, **kw)
    rng = np.random.default_rng(7)
    wc, wb = random_active(rng, mc, mb)
    gc, gb = gpu_vjp(torch, dev, s, cons, blk.bface, wc, wb, dt)
    dc, db = random_active(rng, mc, mb)
    jc, jb = oracle_jvp(orc, cfg, cons, blk.bface, dc, db, dt)
    lhs = np.sum(wc[mc] * jc[mc]) + np.sum(wb[mb] * jb[mb])
    rhs = np.sum(gc[mc] * dc[mc]) + np.sum(gb[mb] * db[mb])
    scale = np.sum(np.abs(wc[mc] * jc[mc])) + np.sum(np.abs(wb[mb] * jb[mb]))
    assert abs(lhs - rhs) <= 1e-12 * scale, (lhs, rhs, scale)
    s.close()


@pytest.mark.parametrize("n,copies", [((5, 3, 7), (40, 1, 1)), ((5, 3, 7), (1, 40, 1)), ((5, 3, 7), (1, 1, 40)),
                                      ((1, 16, 2), (70, 3, 20))])
@pytest.mark.parametrize("integ,recon,rs", SCHEMES)
def test_copies_side_by_side(torch_dev, athmhd, n, copies, integ, recon, rs):  # noqa: F811
    torch, dev = torch_dev
    ng = 2
    blk = inputs.smooth_random(n=n, seed=24, ng=ng)
    rng = np.random.default_rng(9)
    a = (slice(None),) + blk.active
    out = []
    act = [blk.prim[a], blk.bface[a], rng.standard_normal(blk.prim[a].shape), rng.standard_normal(blk.bface[a].shape)]
    for k in ((1, 1, 1), copies):
        N = tuple(n[d] * k[d] for d in range(3))
        s = athmhd.Solver(N, ng, blk.dx, blk.gamma, integrator=integ, recon=recon, riemann=rs, ct_eps=1e-3)
        at = (slice(None),) + tuple(slice(ng, ng + N[d]) for d in (2, 1, 0))
        t = []
        for x, shape in zip(act, (s.cell_shape, s.face_shape) * 2):
            t.append(torch.zeros((x.shape[0],) + shape, dtype=torch.float64, device=dev))
            t[-1][at] = torch.from_numpy(np.tile(x, (1, k[2], k[1], k[0]))).to(dev)
        s.fill_ghosts(t[0], t[1])
        cons = s.prim2cons(t[0], t[1])
        gc, gb = s.step_vjp(cons, t[1], 1e-3, t[2], t[3])
        one = (slice(None),) + tuple(slice(ng, ng + n[d]) for d in (2, 1, 0))
        last = (slice(None),) + tuple(slice(ng + N[d] - n[d], ng + N[d]) for d in (2, 1, 0))
        for w in (one, last):
            out.append((gc[w].cpu().numpy(), gb[w].cpu().numpy()))
        s.close()
    for got in out[1:]:
        for x, y in zip(got, out[0]):
            assert np.abs(x - y).max() <= 1e-13 * np.abs(y).max()
