"""The two ways a coupled mesh without scalars reads its neighbours: in place,
the stages running over the domain, with x3 segments that cross from one layer of
blocks into the next; and from exchanged ghost entries, which a mesh takes
whose layers along x3 hold 4 GiB or more per array (tiny blocks with deep ghost layers
here).  Against the CPU oracle's single block over the domain.

Bar: relative L1 1e-12 per array (that of the other mesh tests)."""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs

pytestmark = pytest.mark.gpu


def _split(torch, x, nblk, mesh):
    """Active entries (nv, L3, L2, L1) of a domain as blocks (nb, nv, n3, n2, n1)."""
    nv = x.shape[0]
    x = x.reshape(nv, mesh[2], nblk[2], mesh[1], nblk[1], mesh[0], nblk[0]).permute(1, 3, 5, 0, 2, 4, 6)
    return x.reshape((-1, nv) + nblk[::-1])


def _join(torch, x, nblk, mesh):
    nv = x.shape[1]
    x = x.reshape((mesh[2], mesh[1], mesh[0], nv) + nblk[::-1]).permute(3, 0, 4, 1, 5, 2, 6)
    return x.reshape(nv, mesh[2] * nblk[2], mesh[1] * nblk[1], mesh[0] * nblk[0])


def _steps(orc, kw, nblk, mesh, ng, floors, steps):
    """Steps of a mesh, whose ghost entries hold NaN at first, and of the oracle."""
    import torch

    from paper_2005_06651_amd import athmhd
    dev = torch.device("cuda:0")
    assert torch.cuda.is_available()
    b = inputs.smooth_random(n=tuple(nblk[d] * mesh[d] for d in range(3)), seed=43, ng=3)
    cfg = orc.cfg_for(b, dfloor=floors[0], pfloor=floors[1], **kw)
    rc, rb = orc.prim2cons(orc.cfg_for(b, **kw), b.prim, b.bface), b.bface.copy()
    s = athmhd.MeshSolver(nblk, mesh, ng, b.dx, b.gamma, **kw)
    s.set_floors(*floors)
    dom = (slice(None),) + b.active
    act = (slice(None), slice(None)) + tuple(slice(ng, ng + nblk[d]) for d in (2, 1, 0))
    tc = torch.full((s.nblocks, 5) + s.cell_shape, float("nan"), dtype=torch.float64, device=dev)
    tf = torch.full((s.nblocks, 3) + s.face_shape, float("nan"), dtype=torch.float64, device=dev)
    for t, x in ((tc, rc), (tf, rb)):
        t[act] = _split(torch, torch.from_numpy(np.ascontiguousarray(x[dom])).to(dev), nblk, mesh)
    layer = mesh[0] * mesh[1] * 8 * tc[0].numel()
    assert (layer >= 2**32) == (ng == 8)
    for _ in range(steps):
        dt, bad = orc.newdt(cfg, rc, rb)
        assert bad == 0
        assert abs(s.newdt(tc, tf) - dt) <= 1e-13 * dt
        assert orc.step(cfg, rc, rb, dt) == 0
        s.step(tc, tf, dt)
    s.newdt(tc, tf)  # raises on a non-physical cell
    s.close()
    for t, y in ((tc, rc[dom]), (tf, rb[dom])):
        x = _join(torch, t[act], nblk, mesh).cpu().numpy()
        for v in range(len(x)):
            assert float(np.abs(x[v] - y[v]).sum()) <= 1e-12 * float(np.abs(y[v]).sum())


CASES = [(dict(integrator="vl2", recon="plm", riemann="hlld"), (0.0, 0.0)),
         (dict(integrator="rk2", recon="plm", riemann="hlle"), (0.8, 0.9)),
         (dict(integrator="rk3", recon="ppm", riemann="hlle"), (0.0, 0.0)),
         (dict(integrator="rk3", recon="ppm", riemann="hlld", ct_eps=1e-3), (0.0, 0.0)),
         (dict(integrator="rk2", recon="dc", riemann="hlle"), (0.8, 0.9))]


@pytest.mark.parametrize("kz", [1, 7, 18])
@pytest.mark.parametrize("kw,floors", CASES)
def test_in_place(orc, monkeypatch, kw, floors, kz):
    monkeypatch.setenv("ATHMHD_KZ", str(kz))
    _steps(orc, kw, (12, 10, 9), (2, 2, 2), 3, floors, 3)


@pytest.mark.parametrize("kw,floors", CASES)
def test_exchanged(orc, kw, floors):
    _steps(orc, kw, (2, 2, 2), (145, 128, 2), 8, floors, 2)
