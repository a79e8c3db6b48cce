"""The work a user has this framework do, as cases to be timed and compared.

Every case is one pass of a user's program through the public entry points of
`paper_2005_06651_amd`: a time step of one periodic block, of a coupled mesh,
of a batch of uneven blocks, the gradient of a rollout, or the refinement and
derefinement of a block.  Sizes are those of the benchmark and the tests; draw
gives others of the same ranges.

  listed()            the cases
  draw(rng)           one more of the same ranges
  prepare(case, seed) what the program holds before the call (on the GPU)
  run(state)          one pass; its outputs
  work(case)          bytes and operations that a pass cannot do without
  exact(case, seed)   the outputs in plain torch, double precision

Inputs come from the seed alone: band-limited random fields given by their
Fourier coefficients, face fields as the curl of a vector potential (exact edge
integrals, so div B is zero to round-off).
"""
import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_2005_06651_amd import athmhd
from paper_2005_06651_amd.rollout import Prim2Cons, Rollout

GAMMA = 5.0 / 3.0
CFL = 0.3
FLOOR = 1e-10
STAGES = {"rk1": 1, "vl2": 2, "rk2": 2, "rk3": 3}


def _dev():
    return torch.device("cuda:0")


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def _block(name, n1, n2, n3, **kw):
    c = dict(name=name, kind="block", n1=n1, n2=n2, n3=n3, field="turbulence", recon="plm", riemann="hlld",
             integrator="vl2", floors=False, scalars=0, charac=False, loop="chain")
    c.update(kw)
    return c


def listed():
    return [
        # a convergence study's small grid: dt to the host every step (newdt, then step), third order
        _block("wave64x32x32", 64, 32, 32, field="wave", recon="ppm", integrator="rk3", loop="host"),
        # one MeshBlock of the usual size by itself: launches and an unfilled chip count
        _block("block64", 64, 64, 64),
        # the benchmark's default workload: decaying turbulence, chained steps
        _block("turbulence256", 256, 256, 256),
        # a box of no particular size: ragged tiles, third order, the simpler Riemann solver, floors
        _block("blast_ragged", 200, 150, 131, field="blast", recon="ppm", riemann="hlle", integrator="rk3",
               floors=True),
        # the largest single block: the strong blast with floors, third order
        _block("blast512", 512, 512, 512, field="blast", recon="ppm", integrator="rk3", floors=True),
        # passive dyes carried along
        _block("dye256", 256, 256, 256, scalars=2),
        # reconstruction on characteristic variables
        _block("charac192", 192, 192, 192, charac=True),
        # one domain as many equal blocks that exchange ghosts
        dict(name="mesh256", kind="mesh", nb=32, m1=8, m2=8, m3=8),
        # a thousand blocks of uneven sizes advanced together, each periodic by itself
        dict(name="batch1024", kind="batch", small=410, middle=410, large=204),
        # blocks of uneven sizes tiling one periodic domain
        dict(name="coupled1032", kind="coupled", cross=192, s16=3, s24=6, s32=6),
        # gradient of a loss after a rollout with respect to the initial state
        dict(name="rollout128", kind="rollout", n1=128, n2=128, n3=128, steps=8),
        # a block refined into its eight children and the children restricted back
        dict(name="refine64", kind="refine", n1=64, n2=64, n3=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["block"] * 5 + ["mesh", "batch", "coupled", "rollout", "refine"])
    if kind == "block":
        c = _block("", _log_int(rng, 12, 300), _log_int(rng, 12, 300), _log_int(rng, 12, 300))
        del c["name"]
        c["field"] = rng.choice(["turbulence", "turbulence", "blast"])
        c["recon"], c["integrator"] = rng.choice([("plm", "vl2"), ("plm", "vl2"), ("plm", "rk2"), ("plm", "rk3"),
                                                  ("ppm", "rk3"), ("ppm", "vl2")])
        c["riemann"] = rng.choice(["hlld", "hlld", "hlle"])
        c["loop"] = rng.choice(["chain", "chain", "host"])
        c["floors"] = c["field"] == "blast"
        option = rng.choice(["", "", "", "scalars", "charac"])
        if option == "scalars":
            c["scalars"] = rng.randint(1, 4)
        c["charac"] = option == "charac"
        return c
    if kind == "mesh":
        return dict(kind="mesh", nb=rng.choice([16, 20, 24, 31, 32, 48, 64]), m1=rng.randint(1, 5),
                    m2=rng.randint(1, 5), m3=rng.randint(1, 5))
    if kind == "batch":
        n = _log_int(rng, 8, 600)
        small, middle = rng.randint(0, n), rng.randint(0, n)
        return dict(kind="batch", small=small, middle=middle, large=rng.randint(1, max(1, n // 2)))
    if kind == "coupled":
        cross = rng.choice([96, 192])
        return dict(kind="coupled", cross=cross, s16=rng.randint(1, 3), s24=rng.randint(1, 4), s32=rng.randint(0, 4))
    if kind == "rollout":
        return dict(kind="rollout", n1=_log_int(rng, 16, 120), n2=_log_int(rng, 16, 120), n3=_log_int(rng, 16, 120),
                    steps=rng.randint(1, 10))
    return dict(kind="refine", n1=2 * _log_int(rng, 8, 60), n2=2 * _log_int(rng, 8, 60), n3=2 * _log_int(rng, 8, 60))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
class _Modes:
    """Real random field sum_k Re(c_k e^{i k.x}) with integer wave vectors
    1 <= |k| <= kmax (in units of 2 pi / box), nb independent ones at once."""

    def __init__(self, rng, nb, kmax):
        self.k = np.arange(-kmax, kmax + 1)
        k1, k2, k3 = np.meshgrid(self.k, self.k, self.k, indexing="ij")
        self.kv = np.stack([k1, k2, k3]).astype(float)
        kk = np.sqrt((self.kv ** 2).sum(0))
        band = (kk >= 1.0) & (kk <= kmax)
        shape = (nb,) + kk.shape
        self.c = np.where(band, rng.standard_normal(shape) + 1j * rng.standard_normal(shape), 0.0)

    def axis(self, n, offset, integral, box):
        """e^{i k x} at x = (i + offset) box / n, or its integral over the cell
        above that point."""
        x = (np.arange(n) + offset) / n
        w = 2.0 * np.pi * self.k[:, None]
        e = np.exp(1j * w * x[None, :])
        if integral:
            h = 1.0 / n
            f = np.where(self.k == 0, h, (np.exp(1j * w[:, 0] * h) - 1.0) / np.where(self.k == 0, 1.0, 1j * w[:, 0]))
            e = e * f[:, None] * box
        return torch.from_numpy(e).to(_dev())

    def field(self, n, offsets=(0.5, 0.5, 0.5), integral=None, box=(1.0, 1.0, 1.0), coef=None):
        """(nb, n3, n2, n1)"""
        c = torch.from_numpy(self.c if coef is None else coef).to(_dev())
        nb, K = c.shape[0], len(self.k)
        e = [self.axis(n[d], offsets[d], integral == d, box[d]) for d in range(3)]
        c = c.reshape(nb * K * K, K) @ e[2]                                       # k1 k2 z
        c = c.reshape(nb, K, K, n[2]).permute(0, 3, 1, 2).reshape(-1, K) @ e[1]   # z k1 y
        c = c.reshape(nb, n[2], K, n[1]).permute(0, 1, 3, 2).reshape(-1, K)       # z y k1
        # the last product in real parts: the largest array is the result
        out = c.real.contiguous() @ e[0].real.contiguous()
        out -= c.imag.contiguous() @ e[0].imag.contiguous()
        return out.reshape(nb, n[2], n[1], n[0])


def _unit(f):
    """f over its largest magnitude, field by field"""
    return f / f.abs().amax(dim=(-3, -2, -1), keepdim=True)


def _curl_faces(A, n, box, rms):
    """Lower-face values (nb, 3, n3, n2, n1) of curl A, A three _Modes, scaled
    to the given rms over all three components."""
    G = []
    for d in range(3):
        off = [0.0, 0.0, 0.0]
        G.append(A[d].field(n, off, integral=d, box=box))
    h = [box[d] / n[d] for d in range(3)]
    B = []
    for d in range(3):
        a, b = (d + 1) % 3, (d + 2) % 3
        B.append(((_up(G[b], a, 1) - G[b]) - (_up(G[a], b, 1) - G[a])) / (h[a] * h[b]))
    B = torch.stack(B, dim=1)
    return B * (rms / B.square().sum(1).mean(dim=(-3, -2, -1)).sqrt())[:, None, None, None, None]


def _up(a, d, o):
    """a at the periodic index + o along direction d (0: x1, the last axis)"""
    return torch.roll(a, -o, dims=-1 - d) if o else a


def _turbulence(rng, n, box, mach=1.0):
    """rho = p = 1, solenoidal velocity at the given rms Mach number, B = 0.5 x
    + curl A with rms(curl A) = 0.1; all fields on 1 <= |k| <= 4."""
    v = [_Modes(rng, 1, 4) for _ in range(3)]
    kv = v[0].kv
    kk = np.maximum((kv ** 2).sum(0), 1.0)
    dot = sum(v[d].c * kv[d] for d in range(3)) / kk
    vel = torch.cat([v[d].field(n, coef=v[d].c - dot * kv[d]) for d in range(3)])
    vel *= mach * math.sqrt(GAMMA) / vel.square().sum(0).mean().sqrt()
    B = _curl_faces([_Modes(rng, 1, 4) for _ in range(3)], n, box, 0.1)[0]
    B[0] += 0.5
    one = torch.ones_like(vel[:1])
    return torch.cat([one, vel, one]), B


def _smooth(rng, nb, n, box, vmax=0.9, low=0.5, high=2.0, kmax=2):
    """nb smooth states: rho, p in [low, high], |v| < vmax, B = B0 + curl A with
    rms(curl A) = 0.2; (nb, 5, ...), (nb, 3, ...)."""
    mid, half = 0.5 * (low + high), 0.5 * (high - low)
    rho = mid + half * _unit(_Modes(rng, nb, kmax).field(n))
    p = mid + half * _unit(_Modes(rng, nb, kmax).field(n))
    vel = torch.stack([_Modes(rng, nb, kmax).field(n) for _ in range(3)], dim=1)
    vel *= vmax / vel.square().sum(1).amax(dim=(-3, -2, -1)).sqrt()[:, None, None, None, None]
    B = _curl_faces([_Modes(rng, nb, kmax) for _ in range(3)], n, box, 0.2)
    B += torch.from_numpy(0.3 * rng.standard_normal((nb, 3))).to(_dev())[:, :, None, None, None]
    return torch.cat([rho[:, None], vel, p[:, None]], dim=1), B


def _blast(rng, n, box):
    """Overpressure sphere of radius 0.1 (p 10 in 0.1) at a random centre, its
    surface smoothed over two cells, in a uniform oblique field."""
    c = rng.random(3)
    h = box[0] / n[0]
    r2 = 0.0
    for d in range(3):
        x = (torch.arange(n[d], dtype=torch.float64, device=_dev()) + 0.5) * (box[d] / n[d])
        dist = (x - c[d] * box[d]).abs()
        dist = torch.minimum(dist, box[d] - dist)
        r2 = r2 + (dist ** 2).reshape([-1 if q == 2 - d else 1 for q in range(3)])
    p = 0.1 + 9.9 * 0.5 * (1.0 - torch.tanh((r2.sqrt() - 0.1) / (2.0 * h)))
    prim = torch.zeros((5,) + tuple(p.shape), dtype=torch.float64, device=_dev())
    prim[0] = 1.0
    prim[4] = p
    B = torch.zeros((3,) + tuple(p.shape), dtype=torch.float64, device=_dev())
    B[:2] = math.sqrt(0.5)
    return prim, B


def _wave(rng, n, box):
    """A linear fast wave (amplitude 1e-6, random phase) along (1, 1, 1) of the
    box in a uniform oblique field."""
    ph = 2.0 * math.pi * rng.random()
    x = [(torch.arange(n[d], dtype=torch.float64, device=_dev()) + 0.5) / n[d] for d in range(3)]
    k = 2.0 * math.pi * torch.tensor([1.0 / b for b in box], dtype=torch.float64)
    phase = 2.0 * math.pi * (x[0][None, None, :] + x[1][None, :, None] + x[2][:, None, None]) + ph
    e = (k / k.norm()).tolist()
    f = torch.cos(phase)
    prim = torch.stack([1.0 + 1e-6 * f, *(2e-6 * e[d] * f for d in range(3)), 1.0 / GAMMA + 1e-6 * f])
    kvec, amp = k.tolist(), 1e-6
    # A = a sin(k.x + ph) across k: closed-form edge integrals
    a = np.cross(np.array([0.3, -0.4, 0.5]), np.array(kvec)) / float(k @ k) * amp
    G = []
    for d in range(3):
        hd = box[d] / n[d]
        xs = [torch.arange(n[q], dtype=torch.float64, device=_dev()) * (box[q] / n[q]) for q in range(3)]
        th = kvec[0] * xs[0][None, None, :] + kvec[1] * xs[1][None, :, None] + kvec[2] * xs[2][:, None, None] + ph
        G.append(a[d] * (torch.cos(th) - torch.cos(th + kvec[d] * hd)) / kvec[d])
    h = [box[d] / n[d] for d in range(3)]
    B = []
    for d in range(3):
        p, q = (d + 1) % 3, (d + 2) % 3
        B.append((1.0, math.sqrt(2.0), 0.5)[d] + ((_up(G[q], p, 1) - G[q]) - (_up(G[p], q, 1) - G[p])) / (h[p] * h[q]))
    return prim, torch.stack(B)


def _dyes(rng, n, count):
    """The first a dye with fronts a few cells wide, the others smooth"""
    f = _unit(_Modes(rng, count, 3).field(n))
    out = 1.0 + 0.9 * f
    out[0] = 0.5 + 0.5 * torch.tanh(f[0] / 0.1)
    return out


def _cut(a, n, origin, ng, extra):
    """Stored array of a block of n cells at origin from a periodic domain's
    active entries a (..., D3, D2, D1), with ng ghost layers (and the padded
    entry of face arrays)"""
    for d in range(3):
        D = a.shape[-1 - d]
        idx = (torch.arange(n[d] + 2 * ng + extra, device=a.device) + origin[d] - ng) % D
        a = a.index_select(a.dim() - 1 - d, idx)
    return a.contiguous()


def _slabs(case):
    """Slab thicknesses along x3 of the coupled layout, mixed"""
    left = {16: case["s16"], 24: case["s24"], 32: case["s32"]}
    out = []
    while any(left.values()):
        for s in (24, 16, 32):
            if left[s]:
                out.append(s)
                left[s] -= 1
    return out


def _layout(case):
    dims, origins, z = [], [], 0
    for s in _slabs(case):
        for y in range(0, case["cross"], s):
            for x in range(0, case["cross"], s):
                dims.append((s, s, s))
                origins.append((x, y, z))
        z += s
    return dims, origins, (case["cross"], case["cross"], z)


def _ng(case):
    return 3 if case.get("recon") == "ppm" else 2


def _widths(case):
    """Cell widths: a box of unit length along x1, cubic cells"""
    return (1.0 / case["n1"],) * 3


def _domain(case, seed):
    """Active primitives and lower faces of the case's periodic domain, and the
    cell widths.  batch: a list of (block size, dx, prims, faces) per size."""
    rng = np.random.default_rng([seed, 20050666])
    kind = case["kind"]
    if kind == "block":
        n, dx = (case["n1"], case["n2"], case["n3"]), _widths(case)
        box = tuple(n[d] * dx[d] for d in range(3))
        make = {"turbulence": _turbulence, "blast": _blast, "wave": _wave}[case["field"]]
        prim, B = make(rng, n, box)
        if case["scalars"]:
            prim = torch.cat([prim, _dyes(rng, n, case["scalars"])])
        return prim, B, dx
    if kind == "mesh":
        n = tuple(case["nb"] * case[m] for m in ("m1", "m2", "m3"))
        dx = (1.0 / n[0],) * 3
        return (*_turbulence(rng, n, tuple(n[d] * dx[d] for d in range(3))), dx)
    if kind == "batch":
        out = []
        for size, count in ((16, case["small"]), (24, case["middle"]), (32, case["large"])):
            if count:
                h = 0.0625 / size
                out.append((size, h, *_smooth(rng, count, (size,) * 3, (0.0625,) * 3)))
        return out
    if kind == "coupled":
        n = _layout(case)[2]
        dx = (1.0 / n[0],) * 3
        prim, B = _smooth(rng, 1, n, tuple(n[d] * dx[d] for d in range(3)))
        return prim[0], B[0], dx
    if kind == "rollout":
        n, dx = (case["n1"], case["n2"], case["n3"]), _widths(case)
        prim, B = _turbulence(rng, n, tuple(n[d] * dx[d] for d in range(3)), mach=0.3)
        target = 1.0 + 0.05 * _unit(_Modes(rng, 1, 4).field(n))[0]
        return prim, B, dx, target
    n, dx = (case["n1"], case["n2"], case["n3"]), _widths(case)
    prim, B = _smooth(rng, 1, n, tuple(n[d] * dx[d] for d in range(3)))
    return prim[0], B[0], dx


def _stored(case, seed):
    """Stored primitives and faces as the program holds them, cell widths"""
    kind, ng = case["kind"], _ng(case)
    if kind == "batch":
        prims, faces, dims, dxs = [], [], [], []
        for size, h, prim, B in _domain(case, seed):
            n = (size,) * 3
            p, f = _cut(prim, n, (0, 0, 0), ng, 0), _cut(B, n, (0, 0, 0), ng, 1)
            prims.append(p)
            faces.append(f)
            dims += [n] * p.shape[0]
            dxs += [(h,) * 3] * p.shape[0]
        return prims, faces, dims, dxs
    prim, B, dx = _domain(case, seed)[:3]
    if kind == "mesh":
        nb = (case["nb"],) * 3
        at = [(x * nb[0], y * nb[1], z * nb[2]) for z in range(case["m3"]) for y in range(case["m2"])
              for x in range(case["m1"])]
        return (torch.stack([_cut(prim, nb, o, ng, 0) for o in at]), torch.stack([_cut(B, nb, o, ng, 1) for o in at]),
                nb, dx)
    if kind == "coupled":
        dims, origins, _ = _layout(case)
        return ([_cut(prim, n, o, ng, 0) for n, o in zip(dims, origins)],
                [_cut(B, n, o, ng, 1) for n, o in zip(dims, origins)], dims, dx)
    n = tuple(prim.shape[-1 - d] for d in range(3))
    return _cut(prim, n, (0, 0, 0), ng, 0), _cut(B, n, (0, 0, 0), ng, 1), n, dx


def _flat(arrays):
    return torch.cat([a.reshape(-1) for a in arrays])


# ---------------------------------------------------------------------------
# The program's state and one pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind, ng = case["kind"], _ng(case)
    if kind == "rollout":
        prim, B, n, dx = _stored(case, seed)
        s = athmhd.Solver(n, ng, dx, GAMMA, recon="plm", riemann="hlld", integrator="vl2", cfl=CFL, ct_eps=1e-3)
        dt = s.newdt(s.prim2cons(prim, B), B)
        return dict(case=case, solver=s, prim=prim, bface=B, dt=dt, target=_domain(case, seed)[3], dV=math.prod(dx))
    if kind == "refine":
        prim, B, n, dx = _stored(case, seed)
        s = athmhd.Solver(n, ng, dx, GAMMA, cfl=CFL)
        cons = s.prim2cons(prim, B)
        return dict(case=case, solver=s, cons=cons, bface=B, fine=[torch.zeros_like(cons) for _ in range(8)],
                    fine_b=[torch.zeros_like(B) for _ in range(8)], back=torch.zeros_like(cons),
                    back_b=torch.zeros_like(B))
    prim, B, n, dx = _stored(case, seed)
    if kind == "block":
        s = athmhd.Solver(n, ng, dx, GAMMA, recon=case["recon"], riemann=case["riemann"],
                          integrator=case["integrator"], cfl=CFL, nscalars=case["scalars"], charac=case["charac"])
        if case["floors"]:
            s.set_floors(FLOOR, FLOOR)
    elif kind == "mesh":
        s = athmhd.MeshSolver(n, (case["m1"], case["m2"], case["m3"]), ng, dx, GAMMA, cfl=CFL)
    elif kind == "batch":
        s = athmhd.BatchSolver(n, dx, ng, GAMMA, cfl=CFL)
        prim, B = _flat(prim), _flat(B)
    else:
        s = athmhd.BatchSolver(n, [dx] * len(n), ng, GAMMA, cfl=CFL)
        s.couple(_layout(case)[1], _layout(case)[2])
        prim, B = _flat(prim), _flat(B)
    cons = s.prim2cons(prim, B)
    if kind == "coupled":
        s.fill_ghosts(cons, B)
    st = dict(case=case, solver=s, cons=cons, bface=B)
    if case.get("loop", "chain") == "chain":
        st["dt"] = torch.tensor([s.newdt(cons, B)], dtype=torch.float64, device=cons.device)
        st["bad"] = torch.zeros(1, dtype=torch.int32, device=cons.device)
    return st


def run(state):
    case, s = state["case"], state["solver"]
    if case["kind"] == "rollout":
        prim = state["prim"].detach().requires_grad_(True)
        cons = Prim2Cons.apply(prim, state["bface"], s)
        cons, bface = Rollout.apply(cons, state["bface"], s, state["dt"], case["steps"])
        loss = ((_inside(cons[0], s.n, s.ng) - state["target"]) ** 2).sum() * state["dV"]
        loss.backward()
        return {"loss": loss.detach(), "cons": cons.detach(), "grad": prim.grad}
    if case["kind"] == "refine":
        octants = [(q & 1, (q >> 1) & 1, q >> 2) for q in range(8)]
        for q, o in enumerate(octants):
            s.prolong(state["cons"], state["bface"], state["fine"][q], state["fine_b"][q], o)
        for q, o in enumerate(octants):
            s.restrict(state["fine"][q], state["fine_b"][q], state["back"], state["back_b"], o)
        return {k: state[k] for k in ("fine", "fine_b", "back", "back_b")}
    if case.get("loop", "chain") == "host":
        dt = s.newdt(state["cons"], state["bface"])
        s.step(state["cons"], state["bface"], dt)
        return {"cons": state["cons"], "bface": state["bface"], "dt": dt}
    s.step_chain(state["cons"], state["bface"], state["dt"], nbad_out=state["bad"])
    return {k: state[k] for k in ("cons", "bface", "dt", "bad")}


# operations of one stage per cell (adds, multiplies, divides, square roots;
# each slope or parabola of a cell once), HLLD; HLLE saves about 300
STAGE_FLOPS = {"dc": 1190.0, "plm": 1370.0, "ppm": 2100.0}


def work(case):
    kind = case["kind"]
    step = STAGE_FLOPS["dc"] + STAGE_FLOPS["plm"]
    if kind == "rollout":
        cells = case["n1"] * case["n2"] * case["n3"]
        # the reverse sweep of an operation costs about twice the operation
        return {"bytes": cells * (64 + 40 + 40), "flops": cells * case["steps"] * 3 * step}
    if kind == "refine":
        coarse = case["n1"] * case["n2"] * case["n3"]
        return {"bytes": coarse * ((9 * 5 + 27) + (9 * 5 + 15)) * 8, "flops": coarse * 400}
    scalars = 0
    if kind == "block":
        cells, scalars = case["n1"] * case["n2"] * case["n3"], case["scalars"]
        per = STAGE_FLOPS[case["recon"]] - (300.0 if case["riemann"] == "hlle" else 0.0)
        if case["integrator"] == "vl2":
            step = STAGE_FLOPS["dc"] - (300.0 if case["riemann"] == "hlle" else 0.0) + per
        else:
            step = STAGES[case["integrator"]] * per
        if case["charac"]:
            step += 3 * 7 * 60 * (1 if case["integrator"] == "vl2" else STAGES[case["integrator"]])
        step += scalars * 60 * STAGES[case["integrator"]]
    elif kind == "mesh":
        cells = case["nb"] ** 3 * case["m1"] * case["m2"] * case["m3"]
    elif kind == "batch":
        cells = case["small"] * 16 ** 3 + case["middle"] * 24 ** 3 + case["large"] * 32 ** 3
    else:
        cells = math.prod(_layout(case)[2])
    # a step reads its state once and writes it once, and yields the next dt
    return {"bytes": cells * (64 + 8 * scalars) * 2, "flops": cells * (step + 100)}


# ---------------------------------------------------------------------------
# The same in plain torch, double precision.  Arrays of active entries only,
# (..., n3, n2, n1), periodic; direction d is axis -1 - d.
# ---------------------------------------------------------------------------
def _cons_of(prim, B):
    """Conserved state of stored primitives (ghosts included) and faces"""
    rho, v, p = prim[..., 0, :, :, :], [prim[..., 1 + d, :, :, :] for d in range(3)], prim[..., 4, :, :, :]
    f = [B[..., d, :, :, :] for d in range(3)]
    lo = [x[..., :-1, :-1, :-1] for x in f]
    bc = [0.5 * (lo[0] + f[0][..., :-1, :-1, 1:]), 0.5 * (lo[1] + f[1][..., :-1, 1:, :-1]),
          0.5 * (lo[2] + f[2][..., 1:, :-1, :-1])]
    e = p / (GAMMA - 1.0) + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2) + 0.5 * (bc[0] ** 2 + bc[1] ** 2 + bc[2] ** 2)
    rows = [rho, rho * v[0], rho * v[1], rho * v[2], e]
    rows += [rho * prim[..., q, :, :, :] for q in range(5, prim.shape[-4])]
    return torch.stack(rows, dim=-4)


def _prims(U, B, floors):
    """rho, v1, v2, v3, p, B1, B2, B3 at cell centres, then C_i; lists of arrays"""
    u = U.unbind(-4)
    b = [0.5 * (x + _up(x, d, 1)) for d, x in enumerate(B.unbind(-4))]
    rho = u[0].clamp(min=FLOOR) if floors else u[0]
    v = [u[1 + d] / rho for d in range(3)]
    p = (GAMMA - 1.0) * (u[4] - 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2) - 0.5 * (b[0] ** 2 + b[1] ** 2 + b[2] ** 2))
    if floors:
        p = p.clamp(min=FLOOR)
    return [rho, *v, p, *b], [u[q] / rho for q in range(5, len(u))]


def _slope(dm, dp):
    pr = dm * dp
    on = pr > 0.0
    return torch.where(on, 2.0 * pr / torch.where(on, dm + dp, 1.0), 0.0)


def _limited(d2, others):
    """The magnitude of d2 and of 1.25 times the others, smallest, where all share a sign"""
    pos, neg, m = d2 > 0.0, d2 < 0.0, d2.abs()
    for o in others:
        pos, neg = pos & (o > 0.0), neg & (o < 0.0)
        m = torch.minimum(m, 1.25 * o.abs())
    return torch.where(pos, m, torch.where(neg, -m, 0.0))


def _ppm_face(qm, q0, q1, q2):
    f = (7.0 / 12.0) * (q0 + q1) - (1.0 / 12.0) * (qm + q2)
    bad = (f - q0) * (q1 - f) < 0.0
    lim = _limited(3.0 * (q0 - 2.0 * f + q1), [qm - 2.0 * q0 + q1, q0 - 2.0 * q1 + q2])
    return torch.where(bad, 0.5 * (q0 + q1) - lim / 6.0, f)


def _edges(q, recon):
    """Left and right edge values of the middle cell of the line q (cells c - r .. c + r)"""
    if recon == "dc":
        return q[0], q[0]
    if recon == "plm":
        s = 0.5 * _slope(q[1] - q[0], q[2] - q[1])
        return q[1] - s, q[1] + s
    a, b, c, d, e = q
    m, p = _ppm_face(a, b, c, d), _ppm_face(b, c, d, e)
    extremum = ((p - c) * (c - m) <= 0.0) | ((b - c) * (c - d) <= 0.0)
    d2 = 6.0 * (m + p) - 12.0 * c
    lim = _limited(d2, [a - 2.0 * b + c, c - 2.0 * d + e, b - 2.0 * c + d])
    r = torch.where(d2 != 0.0, lim / torch.where(d2 != 0.0, d2, 1.0), 0.0)
    dm, dp = m - c, p - c
    p1 = torch.where(dp.abs() >= 2.0 * dm.abs(), c - 2.0 * dm, p)
    m1 = torch.where(dm.abs() >= 2.0 * (p1 - c).abs(), c - 2.0 * (p1 - c), m)
    return torch.where(extremum, c + dm * r, m1), torch.where(extremum, c + dp * r, p1)


REACH = {"dc": 0, "plm": 1, "ppm": 2}


def _face_edges(w, d, recon, charac):
    """Left and right states at the lower D-faces, in the face's frame"""
    a, b = (d + 1) % 3, (d + 2) % 3
    q = [w[0], w[1 + d], w[1 + a], w[1 + b], w[4], w[5 + a], w[5 + b]]
    r = REACH[recon]
    if charac and r:
        lo, hi = _char_edges(q, w[5 + d], d, recon)
    else:
        lo, hi = zip(*[_edges([_up(x, d, o) for o in range(-r, r + 1)], recon) for x in q])
    return [_up(x, d, -1) for x in hi], list(lo)


def _char_edges(q, bn, d, recon):
    """Edges on characteristic variables: differences from the middle cell
    split into its seven waves, limited wave by wave, put together again"""
    r = REACH[recon]
    rho, p, t1, t2 = q[0], q[4], q[5], q[6]
    a2, ca2, bt2 = GAMMA * p / rho, bn * bn / rho, t1 * t1 + t2 * t2
    s = a2 + ca2 + bt2 / rho
    cf2 = 0.5 * (s + (s * s - 4.0 * a2 * ca2).clamp(min=0.0).sqrt())
    cs2 = a2 * ca2 / cf2
    af = ((a2 - cs2) / (cf2 - cs2)).clamp(0.0, 1.0).sqrt()
    as_ = ((cf2 - a2) / (cf2 - cs2)).clamp(0.0, 1.0).sqrt()
    bt = bt2.sqrt()
    e1, e2 = torch.where(bt2 > 0.0, t1 / bt, math.sqrt(0.5)), torch.where(bt2 > 0.0, t2 / bt, math.sqrt(0.5))
    sg = torch.where(bn >= 0.0, 1.0, -1.0)
    a, cf, cs, sr = a2.sqrt(), cf2.sqrt(), cs2.sqrt(), rho.sqrt()
    gp, Q = GAMMA * p, cf2 * af * af + cs2 * as_ * as_

    def waves(dw):
        dpar, dper = e1 * dw[2] + e2 * dw[3], e2 * dw[2] - e1 * dw[3]
        bpar, bper = e1 * dw[5] + e2 * dw[6], e1 * dw[6] - e2 * dw[5]
        fs, ss = af * dw[4] / gp + as_ * bpar / (sr * a), as_ * dw[4] / gp - af * bpar / (sr * a)
        fd, sd = (af * cf * dw[1] - sg * as_ * cs * dpar) / Q, (as_ * cs * dw[1] + sg * af * cf * dpar) / Q
        al = bper / (sg * sr)
        return [0.5 * (fs - fd), 0.5 * (al - dper), 0.5 * (ss - sd), dw[0] - rho * dw[4] / gp, 0.5 * (ss + sd),
                0.5 * (al + dper), 0.5 * (fs + fd)]

    def state(x):
        fs, fd, ss, sd = x[6] + x[0], x[6] - x[0], x[4] + x[2], x[4] - x[2]
        al, dper = x[5] + x[1], x[5] - x[1]
        par, bpar = sg * (af * cf * sd - as_ * cs * fd), sr * a * (as_ * fs - af * ss)
        bper = al * sg * sr
        return [q[0] + x[3] + rho * (af * fs + as_ * ss), q[1] + cf * af * fd + cs * as_ * sd,
                q[2] + e1 * par + e2 * dper, q[3] + e2 * par - e1 * dper, q[4] + gp * (af * fs + as_ * ss),
                q[5] + e1 * bpar - e2 * bper, q[6] + e2 * bpar + e1 * bper]

    line = {o: waves([_up(x, d, o) - x for x in q]) for o in range(-r, r + 1) if o}
    zero = torch.zeros_like(rho)
    lo, hi = zip(*[_edges([line[o][k] if o else zero for o in range(-r, r + 1)], recon) for k in range(7)])
    return state(lo), state(hi)


def _fast(rho, p, bn2, bt2):
    a2 = GAMMA * p / rho
    s = a2 + (bn2 + bt2) / rho
    return (0.5 * (s + (s * s - 4.0 * a2 * bn2 / rho).clamp(min=0.0).sqrt())).sqrt()


def _physical(q, bn):
    """Conserved state and flux in the face's frame: rho, Mn, Mt1, Mt2, E, Bt1, Bt2"""
    rho, vn, v1, v2, p, b1, b2 = q
    pm = 0.5 * (bn * bn + b1 * b1 + b2 * b2)
    e = p / (GAMMA - 1.0) + 0.5 * rho * (vn * vn + v1 * v1 + v2 * v2) + pm
    vb = vn * bn + v1 * b1 + v2 * b2
    U = [rho, rho * vn, rho * v1, rho * v2, e, b1, b2]
    F = [rho * vn, rho * vn * vn + p + pm - bn * bn, rho * vn * v1 - bn * b1, rho * vn * v2 - bn * b2,
         (e + p + pm) * vn - bn * vb, b1 * vn - bn * v1, b2 * vn - bn * v2]
    return U, F


def _hlle(L, R, bn):
    cl, cr = _fast(L[0], L[4], bn * bn, L[5] ** 2 + L[6] ** 2), _fast(R[0], R[4], bn * bn, R[5] ** 2 + R[6] ** 2)
    sl, sr = torch.minimum(L[1] - cl, R[1] - cr), torch.maximum(L[1] + cl, R[1] + cr)
    bp, bm = sr.clamp(min=0.0), sl.clamp(max=0.0)
    (ul, fl), (ur, fr) = _physical(L, bn), _physical(R, bn)
    F = [(bp * a - bm * b + bp * bm * (y - x)) / (bp - bm) for a, b, x, y in zip(fl, fr, ul, ur)]
    return F, torch.maximum(sl.abs(), sr.abs())


def _hlld(L, R, bn):
    cl, cr = _fast(L[0], L[4], bn * bn, L[5] ** 2 + L[6] ** 2), _fast(R[0], R[4], bn * bn, R[5] ** 2 + R[6] ** 2)
    c = torch.maximum(cl, cr)
    sl, sr = torch.minimum(L[1], R[1]) - c, torch.maximum(L[1], R[1]) + c
    smax = torch.maximum(sl.abs(), sr.abs())
    pt = [q[4] + 0.5 * (bn * bn + q[5] ** 2 + q[6] ** 2) for q in (L, R)]
    ml, mr = (sl - L[1]) * L[0], (sr - R[1]) * R[0]
    sm = (mr * R[1] - ml * L[1] - pt[1] + pt[0]) / (mr - ml)
    pts = (mr * pt[0] - ml * pt[1] + ml * mr * (R[1] - L[1])) / (mr - ml)
    sgn = torch.sign(bn)
    side = []
    for q, s, m, P in ((L, sl, ml, pt[0]), (R, sr, mr, pt[1])):
        U, F = _physical(q, bn)
        rs = m / (s - sm)
        den = m * (s - sm) - bn * bn
        flat = den.abs() < 1e-8 * pts
        den = torch.where(flat, 1.0, den)
        c1 = torch.where(flat, 0.0, bn * (sm - q[1]) / den)
        c2 = torch.where(flat, 1.0, (m * (s - q[1]) - bn * bn) / den)
        v1, v2, b1, b2 = q[2] - q[5] * c1, q[3] - q[6] * c1, q[5] * c2, q[6] * c2
        vb, vbs = q[1] * bn + q[2] * q[5] + q[3] * q[6], sm * bn + v1 * b1 + v2 * b2
        es = ((s - q[1]) * U[4] - P * q[1] + pts * sm + bn * (vb - vbs)) / (s - sm)
        side.append(dict(U=U, F=F, s=s, rs=rs, sq=rs.sqrt(), v=(v1, v2), b=(b1, b2), es=es, vbs=vbs,
                         Us=[rs, rs * sm, rs * v1, rs * v2, es, b1, b2]))
    l, r = side
    ssl, ssr = sm - bn.abs() / l["sq"], sm + bn.abs() / r["sq"]
    sq, both = l["sq"] + r["sq"], l["sq"] * r["sq"]
    vd = [(l["sq"] * l["v"][k] + r["sq"] * r["v"][k] + (r["b"][k] - l["b"][k]) * sgn) / sq for k in range(2)]
    bd = [(l["sq"] * r["b"][k] + r["sq"] * l["b"][k] + both * (r["v"][k] - l["v"][k]) * sgn) / sq for k in range(2)]
    vbd = sm * bn + vd[0] * bd[0] + vd[1] * bd[1]
    left = (sl > 0.0) | (~(sr < 0.0) & ((ssl >= 0.0) | (~(ssr <= 0.0) & (sm >= 0.0))))
    star = ~(sl > 0.0) & ~(sr < 0.0)
    double = star & ~(ssl >= 0.0) & ~(ssr <= 0.0) & ~(0.5 * bn * bn < 1e-8 * pts)
    out = []
    Ud = []
    for x, sign in ((l, -1.0), (r, 1.0)):
        ed = x["es"] + sign * x["sq"] * (x["vbs"] - vbd) * sgn
        Ud.append([x["rs"], x["Us"][1], x["rs"] * vd[0], x["rs"] * vd[1], ed, bd[0], bd[1]])
    for k in range(7):
        f = []
        for x, ss, u2 in ((l, ssl, Ud[0]), (r, ssr, Ud[1])):
            y = x["F"][k] + torch.where(star, x["s"] * (x["Us"][k] - x["U"][k]), 0.0)
            f.append(y + torch.where(double, ss * (u2[k] - x["Us"][k]), 0.0))
        out.append(torch.where(left, f[0], f[1]))
    return out, smax


def _rates(U, B, dx, recon, riemann, ct_eps, floors, charac):
    """dU/dt and dB/dt: minus the flux divergence, minus the curl of the corner EMFs"""
    w, C = _prims(U, B, floors)
    dU, emf, wt = [0.0] * (5 + len(C)), {}, []
    for d in range(3):
        a, b = (d + 1) % 3, (d + 2) % 3
        L, R = _face_edges(w, d, recon, charac)
        if floors:
            for q in (L, R):
                q[0], q[4] = q[0].clamp(min=FLOOR), q[4].clamp(min=FLOOR)
        F, smax = (_hlld if riemann == "hlld" else _hlle)(L, R, B[..., d, :, :, :])
        for k, x in zip((0, 1 + d, 1 + a, 1 + b, 4), F):
            dU[k] = dU[k] - (_up(x, d, 1) - x) / dx[d]
        r = REACH[recon]
        for i, c in enumerate(C):
            lo, hi = _edges([_up(c, d, o) for o in range(-r, r + 1)], recon)
            f = F[0] * torch.where(F[0] >= 0.0, _up(hi, d, -1), lo)
            dU[5 + i] = dU[5 + i] - (_up(f, d, 1) - f) / dx[d]
        emf[d, a], emf[d, b] = F[6], -F[5]  # of component a and b, on the D-faces
        if ct_eps > 0.0:
            wt.append((0.5 + 0.5 * F[0] / (0.5 * (L[0] + R[0]) * ct_eps * smax)).clamp(0.0, 1.0))
        else:
            wt.append(0.5 + 0.5 * torch.sign(F[0]))
        del L, R, F, smax
    E = []
    for e in range(3):
        a, b = (e + 1) % 3, (e + 2) % 3
        c0 = -(w[1 + a] * w[5 + b] - w[1 + b] * w[5 + a])
        ca, cb = _up(c0, a, -1), _up(c0, b, -1)
        cab = _up(ca, b, -1)
        ea0, eb0 = emf[a, e], emf[b, e]
        ea1, eb1 = _up(ea0, b, -1), _up(eb0, a, -1)
        wa0, wa1, wb0, wb1 = wt[a], _up(wt[a], b, -1), wt[b], _up(wt[b], a, -1)
        dbp, dbm = wa0 * (ca - eb1) + (1.0 - wa0) * (c0 - eb0), wa1 * (eb1 - cab) + (1.0 - wa1) * (eb0 - cb)
        dap, dam = wb0 * (cb - ea1) + (1.0 - wb0) * (c0 - ea0), wb1 * (ea1 - cab) + (1.0 - wb1) * (ea0 - ca)
        E.append(0.25 * (ea0 + ea1 + eb0 + eb1) + 0.25 * (dbm - dbp) + 0.25 * (dam - dap))
    dB = []
    for d in range(3):
        a, b = (d + 1) % 3, (d + 2) % 3
        dB.append((_up(E[a], b, 1) - E[a]) / dx[b] - (_up(E[b], a, 1) - E[b]) / dx[a])
    return torch.stack(dU, dim=-4), torch.stack(dB, dim=-4)


def _floored(U, B):
    u = list(U.unbind(-4))
    b = [0.5 * (x + _up(x, d, 1)) for d, x in enumerate(B.unbind(-4))]
    u[0] = u[0].clamp(min=FLOOR)
    other = 0.5 * (u[1] ** 2 + u[2] ** 2 + u[3] ** 2) / u[0] + 0.5 * (b[0] ** 2 + b[1] ** 2 + b[2] ** 2)
    u[4] = torch.where((GAMMA - 1.0) * (u[4] - other) >= FLOOR, u[4], FLOOR / (GAMMA - 1.0) + other)
    return torch.stack(u, dim=-4)


def _step(U, B, dt, dx, recon="plm", riemann="hlld", integrator="vl2", ct_eps=0.0, floors=False, charac=False):
    scheme = {"rk1": [(0, 1, 1)], "vl2": [(0, 1, 0.5), (0, 1, 1)], "rk2": [(0, 1, 1), (0.5, 0.5, 0.5)],
              "rk3": [(0, 1, 1), (0.25, 0.75, 0.25), (2 / 3, 1 / 3, 2 / 3)]}[integrator]
    x, y = U, B
    for q, (g0, g1, beta) in enumerate(scheme):
        dU, dB = _rates(x, y, dx, "dc" if integrator == "vl2" and q == 0 else recon, riemann, ct_eps, floors, charac)
        x, y = g0 * x + g1 * U + beta * dt * dU, g0 * y + g1 * B + beta * dt * dB
        if floors:
            x = _floored(x, y)
    return x, y


def _dt_of(U, B, dx, floors=False):
    w, _ = _prims(U, B, floors)
    best = math.inf
    for d in range(3):
        c = _fast(w[0], w[4], w[5 + d] ** 2, w[5 + (d + 1) % 3] ** 2 + w[5 + (d + 2) % 3] ** 2)
        best = min(best, float((dx[d] / (w[1 + d].abs() + c)).min()))
    return CFL * best


def _inside(a, n, ng):
    return a[..., ng:ng + n[2], ng:ng + n[1], ng:ng + n[0]]


def _minmod(a, b):
    return torch.where((a > 0.0) & (b > 0.0), torch.minimum(a, b), torch.where((a < 0.0) & (b < 0.0), torch.maximum(a, b), 0.0))


def _children(U):
    """U (5, n, n, n), periodic: cells of the twice finer grid"""
    s = [_minmod(U - _up(U, d, -1), _up(U, d, 1) - U) for d in range(3)]
    out = torch.empty((U.shape[0],) + tuple(2 * x for x in U.shape[1:]), dtype=U.dtype, device=U.device)
    for q in range(8):
        o = (q & 1, (q >> 1) & 1, q >> 2)
        out[:, o[2]::2, o[1]::2, o[0]::2] = U + 0.25 * sum((2 * o[d] - 1) * s[d] for d in range(3))
    return out


def _child_faces(B):
    """B (3, n, n, n), periodic lower faces: lower faces of the twice finer
    grid (Toth & Roe): each coarse face split by its limited linear profile,
    the faces inside each coarse cell from its divergence and the curl at its
    interior edges"""
    O = []  # O[d][p][q]: the lower coarse face, halves along d + 1, d + 2
    for d in range(3):
        a, b = (d + 1) % 3, (d + 2) % 3
        s = [_minmod(B[d] - _up(B[d], t, -1), _up(B[d], t, 1) - B[d]) for t in (a, b)]
        O.append([[B[d] + 0.25 * ((2 * p - 1) * s[0] + (2 * q - 1) * s[1]) for q in range(2)] for p in range(2)])
    out = torch.empty((3,) + tuple(2 * x for x in B.shape[1:]), dtype=B.dtype, device=B.device)

    def at(d, S, p, q):
        return _up(O[d][p][q], d, S)

    for d in range(3):
        a, b = (d + 1) % 3, (d + 2) % 3
        for p in range(2):
            for q in range(2):
                inner = 0.5 * (at(d, 0, p, q) + at(d, 1, p, q))
                for S in range(2):
                    for i in range(2):
                        sg = 1.0 if S == i else -1.0
                        for k in range(2):
                            inner = inner + sg * (0.1875 if k == q else 0.0625) * at(a, S, k, i)
                            inner = inner + sg * (0.1875 if k == p else 0.0625) * at(b, S, i, k)
                for S, x in ((0, O[d][p][q]), (1, inner)):
                    o = [0, 0, 0]
                    o[d], o[a], o[b] = S, p, q
                    out[d, o[2]::2, o[1]::2, o[0]::2] = x
    return out


def _exact_refine(case, seed):
    prim, B, n, _ = _stored(case, seed)
    ng = _ng(case)
    U = _inside(_cons_of(prim, B), n, ng)
    F = _inside(B, n, ng)
    fU, fF = _children(U), _child_faces(F)
    fine, fine_b = [], []
    for q in range(8):
        o = [n[d] * ((q >> d) & 1) for d in range(3)]
        c, b = torch.zeros_like(prim), torch.zeros_like(B)
        _inside(c, n, ng)[:] = _cut(fU, n, o, 0, 0)
        x = _cut(fF, n, o, 0, 1)
        for d in range(3):  # upper boundary faces along their own direction
            e = [n[k] + (1 if k == d else 0) for k in range(3)]
            _inside(b[d], e, ng)[:] = x[d, :e[2], :e[1], :e[0]]
        fine.append(c)
        fine_b.append(b)
    back, back_b = torch.zeros_like(prim), torch.zeros_like(B)
    _inside(back, n, ng)[:] = fU.reshape(5, n[2], 2, n[1], 2, n[0], 2).mean(dim=(2, 4, 6))
    for d in range(3):
        x = fF[d]
        for t in range(3):
            low = torch.arange(0, 2 * n[t], 2, device=x.device)
            x = x.index_select(2 - t, low) if t == d else 0.5 * (x.index_select(2 - t, low) + x.index_select(2 - t, low + 1))
        x = _cut(x, n, (0, 0, 0), 0, 1)
        e = [n[k] + (1 if k == d else 0) for k in range(3)]
        _inside(back_b[d], e, ng)[:] = x[:e[2], :e[1], :e[0]]
    return {"fine": fine, "fine_b": fine_b, "back": back, "back_b": back_b}


def _exact_rollout(case, seed):
    prim, B, n, dx = _stored(case, seed)
    target = _domain(case, seed)[3]
    ng = _ng(case)
    U0, F = _cons_of(prim, B), _inside(B, n, ng)
    dt = _dt_of(_inside(U0, n, ng), F, dx)
    w = prim.clone().requires_grad_(True)
    x, y = _inside(_cons_of(w, B), n, ng), F

    def one(u, b):
        return _step(u, b, dt, dx, ct_eps=1e-3)

    for _ in range(case["steps"]):
        x, y = checkpoint(one, x, y, use_reentrant=False)
    loss = ((x[0] - target) ** 2).sum() * math.prod(dx)
    loss.backward()
    cons = U0.detach().clone()
    _inside(cons, n, ng)[:] = x.detach()
    return {"loss": loss.detach(), "cons": cons, "grad": w.grad}


def exact(case, seed):
    kind, ng = case["kind"], _ng(case)
    if kind == "refine":
        return _exact_refine(case, seed)
    if kind == "rollout":
        return _exact_rollout(case, seed)
    with torch.no_grad():
        if kind == "batch":
            groups = _domain(case, seed)
            state = []
            for size, h, prim, B in groups:
                n = (size,) * 3
                p, f = _cut(prim, n, (0, 0, 0), ng, 0), _cut(B, n, (0, 0, 0), ng, 1)
                c = _cons_of(p, f)
                state.append((n, (h,) * 3, c, f))
            dt = min(_dt_of(_inside(c, n, ng), _inside(f, n, ng), dx) for n, dx, c, f in state)
            new = math.inf
            for n, dx, c, f in state:
                x, y = _step(_inside(c, n, ng), _inside(f, n, ng), dt, dx)
                _inside(c, n, ng)[:] = x
                _inside(f, n, ng)[:] = y
                new = min(new, _dt_of(x, y, dx))
            cons, bface = _flat([s[2] for s in state]), _flat([s[3] for s in state])
        else:
            prim, B, dx = _domain(case, seed)
            n = tuple(prim.shape[-1 - d] for d in range(3))
            keys = ("recon", "riemann", "integrator", "floors", "charac")
            opt = {k: case[k] for k in keys} if kind == "block" else {}
            floors = bool(opt.get("floors"))
            U = _inside(_cons_of(_cut(prim, n, (0, 0, 0), 1, 0), _cut(B, n, (0, 0, 0), 1, 1)), n, 1).contiguous()
            dt = _dt_of(U, B, dx, floors)
            x, y = _step(U, B, dt, dx, **opt)
            if case.get("loop") == "host":
                new = dt
            else:
                new = _dt_of(x, y, dx, floors)
            if kind == "coupled":  # ghost entries follow the step
                dims, origins, _ = _layout(case)
                cons = _flat([_cut(x, m, o, ng, 0) for m, o in zip(dims, origins)])
                bface = _flat([_cut(y, m, o, ng, 1) for m, o in zip(dims, origins)])
            elif kind == "mesh":  # ghost entries stay as they were
                m = (case["nb"],) * 3
                at = [(i * m[0], j * m[1], k * m[2]) for k in range(case["m3"]) for j in range(case["m2"])
                      for i in range(case["m1"])]
                cons = torch.stack([_cut(U, m, o, ng, 0) for o in at])
                bface = torch.stack([_cut(B, m, o, ng, 1) for o in at])
                for q, o in enumerate(at):
                    _inside(cons[q], m, ng)[:] = _cut(x, m, o, 0, 0)
                    _inside(bface[q], m, ng)[:] = _cut(y, m, o, 0, 0)
            else:
                cons, bface = _cut(U, n, (0, 0, 0), ng, 0), _cut(B, n, (0, 0, 0), ng, 1)
                _inside(cons, n, ng)[:] = x
                _inside(bface, n, ng)[:] = y
        out = {"cons": cons, "bface": bface, "dt": new if case.get("loop") == "host" else torch.tensor([new], dtype=torch.float64)}
        if case.get("loop", "chain") == "chain":
            out["bad"] = torch.zeros(1, dtype=torch.int32)
        return out
