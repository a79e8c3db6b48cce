"""The CFL reduction of a two-level composite takes two launches, the second of
which finishes it.  An error that ends newdt between them leaves nothing of it to
the next one."""
import ctypes as C

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


def test_reduction_after_a_reported_error(athmhd, orc):
    """A HIP error left pending by other code of the process is reported by
    the next launch: newdt of a two-level composite raises after the first of its
    two launches.  The next newdt is that of its own state."""
    import torch
    dev = torch.device("cuda:0")
    n, ng = (8, 8, 8), 2
    box = (2.0, 1.0, 1.0)
    cg = inputs.analytic_state((2 * n[0], n[1], n[2]), ng, box, seed=3)
    fg = inputs.analytic_state((4 * n[0], 2 * n[1], 2 * n[2]), ng, box, seed=3)
    prim, face = inputs.two_level(cg, fg, n)
    face = np.ascontiguousarray(face)
    cfg = orc.make_cfg(n, ng, cg.dx, cg.gamma)
    s = athmhd.TwoLevelSolver(n, ng, cg.dx, cg.gamma)
    tf = torch.from_numpy(face).to(dev)
    states = []
    for v in (0.0, 5.0):
        w = np.ascontiguousarray(prim)
        w[:, 1] += v
        states.append(torch.from_numpy(np.stack([orc.prim2cons(cfg, w[q], face[q]) for q in range(9)])).to(dev))
    slow, fast = states
    want = s.newdt(slow, tf)
    dt = s.newdt(fast, tf)
    assert dt < 0.8 * want
    assert athmhd.lib().hipSetDevice(C.c_int(1 << 20)) != 0
    with pytest.raises(athmhd.AthmhdError):
        s.newdt(fast, tf)
    dt = s.newdt(slow, tf)
    assert dt == want
    s.close()
