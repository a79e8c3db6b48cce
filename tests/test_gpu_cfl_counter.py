"""The CFL reduction is finished by the last of its workgroups, which an atomic
count names, and prepared by the one before it: nothing clears it in between.
So a large non-physical count may not leave it half done."""
import numpy as np
import pytest

from paper_2005_06651_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def athmhd():
    import torch

    from paper_2005_06651_amd import athmhd as A
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    A.lib()
    return A


def test_reduction_with_a_count_past_2_31(athmhd):
    """Chained steps of a state without a physical cell, whose count stays in
    the handle (nbad_out not given) and grows by at least a cell each per step:
    past 2^31 newdt still reports it, and the reductions after that are those of
    a new handle, for a state with another limit than the last good one."""
    import torch
    dev = torch.device("cuda:0")
    n = (256, 256, 256)
    good = inputs.uniform(n=n, ng=2, v=(0.3, -0.2, 0.1))
    fast = inputs.uniform(n=n, ng=2, v=(3.0, -0.2, 0.1))
    kw = dict(integrator="rk1", recon="dc", riemann="hlle")
    s = athmhd.Solver(n, 2, good.dx, good.gamma, **kw)
    face = torch.from_numpy(good.bface).to(dev)
    slow_c = s.prim2cons(torch.from_numpy(good.prim).to(dev), face)
    fast_c = s.prim2cons(torch.from_numpy(fast.prim).to(dev), face)
    fresh = athmhd.Solver(n, 2, good.dx, good.gamma, **kw)
    want_slow, want_fast = fresh.newdt(slow_c, face), fresh.newdt(fast_c, face)
    fresh.close()
    assert want_fast < 0.5 * want_slow
    assert s.newdt(slow_c, face) == want_slow
    bad_c, bad_f = slow_c.clone(), face.clone()
    bad_c[0] = -1.0
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device=dev)
    steps = 2**31 // (n[0] * n[1] * n[2]) + 4
    for _ in range(steps):
        s.step_chain(bad_c, bad_f, dt)
    assert np.isinf(dt.item())  # no cell gives a limit
    with pytest.raises(athmhd.NonPhysicalState):
        s.newdt(fast_c, face)
    assert s.newdt(fast_c, face) == want_fast
    assert s.newdt(slow_c, face) == want_slow
    dt.fill_(1e-9)
    nbad = torch.full((1,), -1, dtype=torch.int32, device=dev)
    s.step_chain(fast_c, face, dt, nbad)
    assert nbad.item() == 0 and abs(dt.item() - want_fast) <= 1e-6 * want_fast
    s.close()
