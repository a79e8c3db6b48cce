"""athmhd_floor_count is a number of the states: a stage counts each active
cell and each face state once, however its kernels are planned (x3 segments, thread
tiles, one block or many, a mesh or a batch)."""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs

pytestmark = pytest.mark.gpu

N, NG = (37, 26, 10), 3


def _floored(s, cons, face, steps):
    """Steps of a solver on this state with floors; the activations."""
    import torch
    dev = torch.device("cuda:0")
    s.set_floors(0.8, 0.9)
    tc, tb = torch.from_numpy(cons).to(dev), torch.from_numpy(face).to(dev)
    s.floor_count()
    for _ in range(steps):
        s.step(tc, tb, 1e-3)
    n = s.floor_count()
    s.close()
    return n


@pytest.fixture(scope="module")
def state(orc):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    b = inputs.smooth_random(n=N, seed=27, ng=NG)
    return b, orc.prim2cons(orc.cfg_for(b), b.prim, b.bface), b.bface


@pytest.mark.parametrize("integ,recon,steps", [("vl2", "plm", 2), ("rk1", "dc", 2)])
def test_count_is_independent_of_the_plan(state, monkeypatch, integ, recon, steps):
    from paper_2005_06651_amd import athmhd
    b, cons, face = state
    kw = dict(integrator=integ, recon=recon, riemann="hlle")
    counts = {}
    for kz in (None, 1, 3, 10):
        if kz:
            monkeypatch.setenv("ATHMHD_KZ", str(kz))
        for nb in (1, 40, 300):
            c, f = (np.broadcast_to(x, (nb,) + x.shape).copy() for x in (cons, face))
            s = athmhd.Solver(N, NG, b.dx, b.gamma, nblocks=nb, **kw)
            counts[kz, nb] = _floored(s, c, f, steps) / nb
    monkeypatch.delenv("ATHMHD_KZ")
    for mesh, n in (((1, 2, 2), (37, 13, 5)), ((1, 1, 5), (37, 26, 2))):
        mc, mf = inputs.split_mesh(cons, face, NG, n, mesh)
        s = athmhd.MeshSolver(n, mesh, NG, b.dx, b.gamma, **kw)
        counts[mesh] = _floored(s, mc, mf, steps)
    s = athmhd.BatchSolver([N, N], [b.dx, b.dx], NG, b.gamma, **kw)
    counts["batch"] = _floored(s, inputs.pack([cons, cons]), inputs.pack([face, face]), steps) / 2
    want = counts[None, 1]
    assert want > 0 and set(counts.values()) == {want}, counts


@pytest.mark.parametrize("charac", [False, True])
def test_count_is_independent_of_the_segments(state, monkeypatch, charac):
    """PPM and characteristic PLM in one kernel: on a plateau of floored cells
    their face states lie on the floor up to rounding, which other kernels may do
    otherwise."""
    from paper_2005_06651_amd import athmhd
    b, cons, face = state
    counts = []
    for kz in (1, 3, 4, 10):
        monkeypatch.setenv("ATHMHD_KZ", str(kz))
        c, f = (np.broadcast_to(x, (300,) + x.shape).copy() for x in (cons, face))
        s = athmhd.Solver(N, NG, b.dx, b.gamma, nblocks=300, integrator="rk1", recon="plm" if charac else "ppm",
                          riemann="hlle", charac=charac)
        counts.append(_floored(s, c, f, 1))
    assert counts[0] > 0 and counts[0] % 300 == 0 and len(set(counts)) == 1, counts


def test_count_of_a_uniform_state(state):
    """Below the density floor everywhere: a donor-cell stage counts every cell
    once, and the floor pass after it once again; the face states, formed of
    floored primitives, lie on the floor."""
    from paper_2005_06651_amd import athmhd
    b, _, _ = state
    u = inputs.uniform(n=N, ng=NG, rho=0.5, p=1.0, dx=b.dx)
    s = athmhd.Solver(N, NG, u.dx, u.gamma, integrator="rk1", recon="dc", riemann="hlle")
    cons = np.empty((5,) + u.prim.shape[1:])
    cons[0] = u.prim[0]
    cons[1:4] = u.prim[0] * u.prim[1:4]
    cons[4] = u.prim[4] / (u.gamma - 1.0) + 0.5 * u.prim[0] * (u.prim[1:4] ** 2).sum(0) + \
        0.5 * sum(u.bface[d].flat[0] ** 2 for d in range(3))
    cells = N[0] * N[1] * N[2]
    count = _floored(s, cons, u.bface, 1)
    assert count == 2 * cells
