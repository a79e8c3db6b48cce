"""Reverse mode at sizes where the layout of its scratch and the order of its
workgroups change: from 4096 cells the arrays lie an odd number of 256-byte
lines apart, and from 4096 cells in a plane each XCD runs several neighbouring
workgroups (with a remainder group whose last threads have no cell).  Lines of
faces are laid end to end over workgroups that complete 61 or 63 cells of them
along x1 and 29 or 15 (8 or 16 cells of x1 side by side) along x2 and x3: the
last sizes put line ends and workgroup ends at and beside each other.

Oracle: the transposition identity <w, J d> = <J^T w, d> with the CPU oracle's
exact directional derivatives; both sides are sums of rounded products, whose
relative error against the sum of their magnitudes stays far below 1e-12.
"""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs
from test_gpu_adjoint import active_masks, athmhd, gpu_vjp, oracle_jvp, random_active, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [(16, 16, 15), (16, 16, 16), (33, 17, 9), (64, 64, 3), (131, 65, 4),
         (61, 9, 29), (63, 29, 12), (8, 30, 26), (17, 15, 61), (2, 3, 64), (1, 1, 5)]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("integ,recon,rs", [("vl2", "plm", "hlld"), ("rk1", "plm", "hlle"), ("rk1", "dc", "hlld")])
def test_transposition_over_layouts(torch_dev, athmhd, orc, n, integ, recon, rs):  # noqa: F811
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
    for _ in range(2):
        dc, db = random_active(rng, mc, mb)
        jc, jb = oracle_jvp(orc, cfg, cons, blk.bface, dc, db, dt)
        lhs = np.sum(wc[mc] * jc[mc]) + np.sum(wb[mb] * jb[mb])
        rhs = np.sum(gc[mc] * dc[mc]) + np.sum(gb[mb] * db[mb])
        scale = np.sum(np.abs(wc[mc] * jc[mc])) + np.sum(np.abs(wb[mb] * jb[mb]))
        assert abs(lhs - rhs) <= 1e-12 * scale, (lhs, rhs, scale)
    s.close()


def test_blocks_of_a_padded_layout(torch_dev, athmhd, orc):  # noqa: F811
    """Two blocks at once equal each by itself, bit by bit."""
    torch, dev = torch_dev
    blocks = [inputs.smooth_random(n=(33, 17, 9), seed=40 + b, ng=2) for b in range(2)]
    b0 = blocks[0]
    kw = dict(integrator="vl2", recon="plm", riemann="hlld", ct_eps=1e-3)
    cfg = orc.cfg_for(b0, **kw)
    cons = [orc.prim2cons(cfg, b.prim, b.bface) for b in blocks]
    mc, mb = active_masks(b0.n, b0.ng)
    rng = np.random.default_rng(8)
    w = [random_active(rng, mc, mb) for _ in blocks]
    two = athmhd.Solver(b0.n, b0.ng, b0.dx, b0.gamma, nblocks=2, **kw)
    gc, gb = gpu_vjp(torch, dev, two, np.stack(cons), np.stack([b.bface for b in blocks]),
                     np.stack([x for x, _ in w]), np.stack([y for _, y in w]), 1e-3)
    one = athmhd.Solver(b0.n, b0.ng, b0.dx, b0.gamma, **kw)
    for q, b in enumerate(blocks):
        c1, f1 = gpu_vjp(torch, dev, one, cons[q], b.bface, w[q][0], w[q][1], 1e-3)
        assert np.array_equal(gc[q], c1) and np.array_equal(gb[q], f1)
    two.close()
    one.close()
