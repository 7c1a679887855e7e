"""Performance cases of the library: what a user's program has it do, through
the public Python entry points (Sim, Batch, ParticleSim, autograd.evolve),
from the smallest boxes to the largest ones of the benchmark.

listed() gives the cases, draw(rng) one more of the same ranges, prepare()
what a program holds before the call, run() one pass, work() the bytes and
operations the pass needs at least, exact() the same outputs from a plain
torch float64 evaluation of the method.

A pass of a box advances it by a few Runge-Kutta steps and reads the state
(or the diagnostics) back, as a program does between two outputs; the next
pass continues from there.  Launch shapes are the library's built-in ones.
"""
import math

import numpy as np
import torch
import torch.utils.checkpoint

from paper_2101_02745_amd import autograd as A
from paper_2101_02745_amd import inputs as I
from paper_2101_02745_amd._lib import HostConfig
from paper_2101_02745_amd.particles import ParticleSim
from paper_2101_02745_amd.sim import Batch, Sim

# cell width and time step of the paper's fiducial 1D box (64 pi over 2048
# cells), of the batch and general-placement boxes, of the small test box,
# and of the 3D boxes
FIDUCIAL = dict(dx=64.0 * math.pi / 2048, dt=0.1)
COARSE = dict(dx=0.2, dt=0.1)
SMALL = dict(dx=2.0, dt=0.2)
CUBE = dict(dx=1.0, dt=0.2)


def listed():
    return [
        # the smallest run (tests, examples, a scan of many tiny boxes one by
        # one): 832 particles, all latency
        dict(name="box_32x26", kind="box", nx=1, ny=1, nz=32, ndir=26, shape=1, steps=10,
             start="seeds", output="state", **SMALL),
        # following a small box in time: single steps, diagnostics after each
        dict(name="monitor_200x92", kind="box", nx=1, ny=1, nz=200, ndir=92, shape=1, steps=1,
             start="seeds", output="diagnostics", **COARSE),
        # ragged mid-size 1D box with the quadratic shape function and matter
        dict(name="box_777x92_quadratic", kind="box", nx=1, ny=1, nz=777, ndir=92, shape=2,
             steps=10, start="saturated", output="state", matter=True, **COARSE),
        # the headline 1D box of the benchmark, between two snapshots
        dict(name="box_2048x378", kind="box", nx=1, ny=1, nz=2048, ndir=378, shape=1, steps=10,
             start="seeds", output="state", **FIDUCIAL),
        # a parameter study: 24 uneven 1D boxes advanced together
        dict(name="batch_24", kind="batch", nsim=24, nz_lo=256, nz_hi=4096, shape=1, steps=4,
             start="seeds", **COARSE),
        # gradients of the final flavor content (forward and backward)
        dict(name="adjoint_512x128", kind="adjoint", nz=512, ndir=128, shape=1, steps=40, ckpt=20,
             **COARSE),
        # the 3D box of the benchmark
        dict(name="box_64x64x64x92", kind="box", nx=64, ny=64, nz=64, ndir=92, shape=1, steps=2,
             start="seeds", output="state", **CUBE),
        # a ragged 3D box with the paper's quadratic shape function
        dict(name="box_50x44x36x24_quadratic", kind="box", nx=50, ny=44, nz=36, ndir=24, shape=2,
             steps=4, start="saturated", output="state", **CUBE),
        # 3D rows longer than a wave
        dict(name="box_150x40x32x24", kind="box", nx=150, ny=40, nz=32, ndir=24, shape=1, steps=4,
             start="saturated", output="state", **CUBE),
        # general placement: a small box, the 1D box and the 3D box of the
        # benchmark (exact sums, the default)
        dict(name="particles_64x16", kind="particles", nx=1, ny=1, nz=64, ppc=16, ndir=26, shape=1,
             steps=10, exact=True, start="seeds", **COARSE),
        dict(name="particles_2048x378", kind="particles", nx=1, ny=1, nz=2048, ppc=378, ndir=378,
             shape=1, steps=8, exact=True, start="seeds", **FIDUCIAL),
        dict(name="particles_32x32x32x92", kind="particles", nx=32, ny=32, nz=32, ppc=92, ndir=92,
             shape=1, steps=4, exact=True, start="seeds", **CUBE),
    ]


NDIRS = (6, 24, 26, 64, 92, 128, 378)   # direction counts of the tests and the paper's tables


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _ndir(rng, most=378):
    if rng.random() < 0.3:
        return 2 * rng.randint(3, most // 2)    # any even count
    return rng.choice([d for d in NDIRS if d <= most])


def draw(rng):
    kind = rng.choice(["box1d", "box1d", "box1d", "box3d", "box3d", "batch", "adjoint", "particles1d",
                       "particles1d", "particles3d"])
    start = rng.choice(["seeds", "saturated"])
    if kind == "box1d":
        g = rng.choice([FIDUCIAL, COARSE, SMALL])
        ndir = _ndir(rng)
        nz = _log(rng, 20, 5000)
        return dict(kind="box", nx=1, ny=1, nz=nz, ndir=ndir, shape=rng.choice([1, 1, 2]),
                    steps=rng.randint(1, 16), start=start,
                    output=rng.choice(["state", "state", "diagnostics"]),
                    matter=rng.random() < 0.3, **g)
    if kind == "box3d":
        ndir = rng.choice([6, 24, 26, 92])
        most = 1.5e6 / ndir
        nx = _log(rng, 8, 160)
        ny = _log(rng, 4, max(4, min(64, most / nx / 4)))
        nz = _log(rng, 4, max(4, min(64, most / nx / ny)))
        return dict(kind="box", nx=nx, ny=ny, nz=nz, ndir=ndir, shape=rng.choice([1, 1, 2]),
                    steps=rng.randint(1, 6), start=start, output="state", **CUBE)
    if kind == "batch":
        lo = _log(rng, 40, 400)
        return dict(kind="batch", nsim=rng.randint(3, 24), nz_lo=lo, nz_hi=lo * rng.randint(2, 8),
                    shape=rng.choice([1, 1, 2]), steps=rng.randint(1, 8), start=start, **COARSE)
    if kind == "adjoint":
        return dict(kind="adjoint", nz=_log(rng, 32, 900), ndir=_ndir(rng, 128),
                    shape=rng.choice([1, 1, 2]), steps=rng.randint(5, 40), ckpt=rng.choice([5, 10, 20]),
                    **rng.choice([FIDUCIAL, COARSE]))
    if kind == "particles1d":
        return dict(kind="particles", nx=1, ny=1, nz=_log(rng, 32, 2048), ppc=_log(rng, 8, 400),
                    ndir=_ndir(rng), shape=rng.choice([1, 1, 2]), steps=rng.randint(1, 12),
                    exact=rng.random() < 0.75, start=start, **rng.choice([FIDUCIAL, COARSE]))
    return dict(kind="particles", nx=rng.randint(8, 24), ny=rng.randint(8, 24), nz=rng.randint(8, 24),
                ppc=_log(rng, 8, 100), ndir=rng.choice([24, 26, 92]), shape=rng.choice([1, 1, 2]),
                steps=rng.randint(1, 6), exact=rng.random() < 0.75, start=start, **CUBE)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
DEV = "cuda:0"


def _gen(seed, stream=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + stream)
    return g


def _uniform(shape, g):
    return 2.0 * torch.rand(shape, dtype=torch.float64, device=DEV, generator=g) - 1.0


def _state(case, n, seed, stream=0):
    """[18][n]: the paper's initial condition (electron flavor with small
    random off-diagonal seeds), or pure states in any direction of flavor
    space, as after the instability has saturated."""
    g = _gen(seed, stream)
    s = torch.zeros((18, n), dtype=torch.float64, device=DEV)
    if case["start"] == "seeds":
        for o in (0, 9):
            u = 1e-6 * _uniform((4, n), g)
            s[o + 3:o + 7] = u
            s[o + 1] = u[0] * u[0] + u[1] * u[1]
            s[o + 2] = u[2] * u[2] + u[3] * u[3]
            s[o] = 1.0 - s[o + 1] - s[o + 2]
        return s
    for o in (0, 9):
        p = torch.randn((6, n), dtype=torch.float64, device=DEV, generator=g)
        p /= p.square().sum(0).sqrt()
        for k in range(3):
            s[o + k] = p[2 * k] ** 2 + p[2 * k + 1] ** 2
        for k, (a, b) in zip((3, 5, 7), ((0, 1), (0, 2), (1, 2))):
            s[o + k] = p[2 * a] * p[2 * b] + p[2 * a + 1] * p[2 * b + 1]
            s[o + k + 1] = p[2 * a + 1] * p[2 * b] - p[2 * a] * p[2 * b + 1]
    return s


def _angles(seed):
    """nbar/n, f, fbar and the flux axis of a box, from the seed."""
    u = np.random.RandomState(int(seed) % (1 << 31)).rand(4)
    ang = math.radians(90.0 * u[3])
    return 0.5 + u[0], -0.4 + 0.8 * u[1], -0.4 + 0.8 * u[2], (math.sin(ang), 0.0, math.cos(ang))


def _workload(case, seed, nz=None, ndir=None):
    nbar, f, fbar, nhat = _angles(seed)
    n = (case.get("nx", 1), case.get("ny", 1), nz or case["nz"])
    dx = case["dx"]
    length = tuple(1.0 if n[a] == 1 else n[a] * dx for a in range(3))
    return I.Workload(name="case", ncell=n, length=length, ndir=ndir or case["ndir"], dt=case["dt"],
                      steps=case["steps"], nbar_over_n=nbar, f=f, fbar=fbar, nhat=nhat,
                      vmat=(2.0, 0.5, 0.1) if case.get("matter") else (0.0, 0.0, 0.0),
                      shape_order=case["shape"])


def _batch_boxes(case, seed):
    """The boxes of a batch: cell counts and direction counts are the case's
    own (the same for every seed), densities and fluxes the seed's."""
    r = np.random.RandomState(77 + case["nsim"] + case["nz_lo"])
    out = []
    for i in range(case["nsim"]):
        nz = int(r.randint(case["nz_lo"], case["nz_hi"] + 1))
        ndir = (64, 128, 378)[int(r.randint(3))]
        out.append(_workload(case, 1000 * (int(seed) % 1000003) + i, nz, ndir))
    return out


def _particles(case, seed):
    nbar, f, fbar, nhat = _angles(seed)
    n = (case["nx"], case["ny"], case["nz"])
    length = tuple(1.0 if n[a] == 1 else n[a] * case["dx"] for a in range(3))
    return I.ParticleWorkload(name="case", ncell=n, length=length, ppc=case["ppc"], ndir=case["ndir"],
                              dt=case["dt"], steps=case["steps"], nbar_over_n=nbar, f=f, fbar=fbar,
                              nhat=nhat, shape_order=case["shape"])


def _particle_arrays(case, w, seed):
    """Positions [np][3] (uniform over the box), directions, weights (N,
    Nbar) and state, on the device."""
    n = w.nparticles
    pos = torch.rand((n, 3), dtype=torch.float64, device=DEV, generator=_gen(seed, 5))
    pos *= torch.tensor(w.length, dtype=torch.float64, device=DEV)
    table = I.directions(w.ndir)
    N, Nb = I.particle_weights(table, w.dV, 1.0, w.f, w.nbar_over_n, w.fbar, w.nhat)
    d = torch.arange(n, device=DEV) % w.ndir
    at = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)[d]  # noqa: E731
    scale = w.ndir / w.ppc
    return pos, at(table), at(N) * scale, at(Nb) * scale, _state(case, n, seed)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "box":
        w = _workload(case, seed)
        sim = Sim.from_workload(w, device=DEV)
        sim.set_state(_state(case, w.nparticles, seed).reshape(18, w.ndir, w.ncell_total))
        return dict(case=case, sim=sim)
    if kind == "batch":
        ws = _batch_boxes(case, seed)
        b = Batch([HostConfig.from_workload(w) for w in ws], device=DEV)
        for i, w in enumerate(ws):
            b.set_state(i, _state(case, w.nparticles, seed, i).reshape(18, w.ndir, w.ncell_total))
        return dict(case=case, batch=b)
    if kind == "adjoint":
        w = _workload(case, seed)
        return dict(case=case, w=w, params=_adjoint_params(w), seeds=_adjoint_seeds(w, seed))
    w = _particles(case, seed)
    ps = ParticleSim.from_workload(w, device=DEV, exact=case["exact"])
    ps.set(*_particle_arrays(case, w, seed))
    return dict(case=case, sim=ps)


def _adjoint_params(w):
    return torch.tensor([w.nbar_over_n, w.f, w.fbar], dtype=torch.float64, device=DEV)


def _adjoint_seeds(w, seed):
    return 1e-3 * _uniform((8, w.ndir, w.ncell_total), _gen(seed))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        b = state["batch"]
        b.step(case["steps"])
        return [b.get_state(i) for i in range(b.nsim)]
    if kind == "adjoint":
        p = state["params"].detach().requires_grad_(True)
        s = state["seeds"].detach().requires_grad_(True)
        nu, nubar = A.evolve(p, s, state["w"], case["steps"], ckpt_every=case["ckpt"])
        (nu + 0.5 * nubar).backward()
        return dict(nu=nu, nubar=nubar, params=p.grad, seeds=s.grad)
    sim = state["sim"]
    sim.step(case["steps"])
    if case.get("output") == "diagnostics":
        m = sim.moments()
        return dict(moments=m, averages=sim.domain_averages(m), totals=sim.flavor_totals(),
                    trace=sim.check(1e-6) < 1e-6)
    return sim.get_state()


# ---------------------------------------------------------------------------
# work: the state read and written once per step (and read for the output),
# the operations of the four Runge-Kutta stages
# ---------------------------------------------------------------------------
def _flops(nparticle, ndim, shape):
    corners = (shape + 1) ** ndim
    # per stage: gather and deposit of 4 moment groups of 9 reals, H and Hbar,
    # two commutators, stage updates
    return 4.0 * nparticle * (2 * 72 * corners + 54 + 18 + 2 * 100 + 72)


def work(case):
    kind = case["kind"]
    ndim = 3 if case.get("nx", 1) > 1 else 1
    if kind == "batch":
        n = sum(w.nparticles for w in _batch_boxes(case, 0))
    elif kind == "particles":
        n = case["nx"] * case["ny"] * case["nz"] * case["ppc"]
    else:
        n = case.get("nx", 1) * case.get("ny", 1) * case["nz"] * case["ndir"]
    steps = case["steps"]
    if kind == "adjoint":
        # the forward pass and its reversal, each reading and writing a state
        return dict(bytes=2 * 288.0 * n * steps, flops=3 * steps * _flops(n, ndim, case["shape"]))
    each = 288.0 + (2 * 64.0 if kind == "particles" else 0.0)
    return dict(bytes=n * (each * steps + 288.0), flops=steps * _flops(n, ndim, case["shape"]))


# ---------------------------------------------------------------------------
# exact: the same method in plain torch, float64, particle by particle
# ---------------------------------------------------------------------------
UP = ((0, 1), (0, 2), (1, 2))


def _unpack(p):
    """Nine packed reals [9][n] -> 3x3 lists of complex tensors."""
    m = [[None] * 3 for _ in range(3)]
    for k in range(3):
        m[k][k] = torch.complex(p[k], torch.zeros_like(p[k]))
    for q, (a, b) in enumerate(UP):
        m[a][b] = torch.complex(p[3 + 2 * q], p[4 + 2 * q])
        m[b][a] = m[a][b].conj()
    return m


def _pack(m):
    return torch.stack([m[0][0].real, m[1][1].real, m[2][2].real]
                       + [part for a, b in UP for part in (m[a][b].real, m[a][b].imag)])


def _bracket(h, r):
    """-i [H, rho], packed, for Hermitian H and rho (packed)."""
    H, R = _unpack(h), _unpack(r)
    C = [[H[a][0] * R[0][b] + H[a][1] * R[1][b] + H[a][2] * R[2][b] for b in range(3)] for a in range(3)]
    return _pack([[-1j * (C[a][b] - C[b][a].conj()) for b in range(3)] for a in range(3)])


CONJ = (1.0, 1.0, 1.0, 1.0, -1.0, 1.0, -1.0, 1.0, -1.0)


class _Plain:
    """A periodic box of particles: pos, v [3][n], weights per volume."""

    def __init__(self, ncell, dx, pos, v, wN, wNb, hvac, vmat, dt, shape):
        self.n, self.dx, self.pos, self.v = ncell, dx, pos, v
        self.wN, self.wNb, self.dt, self.shape = wN, wNb, dt, shape
        h = [hvac[0, 0].real, hvac[1, 1].real, hvac[2, 2].real]
        for a, b in UP:
            h += [hvac[a, b].real, hvac[a, b].imag]
        self.hvac = torch.tensor(h, dtype=torch.float64, device=DEV)[:, None]
        self.vmat = torch.tensor(list(vmat) + [0.0] * 6, dtype=torch.float64, device=DEV)[:, None]
        self.sign = torch.tensor(CONJ, dtype=torch.float64, device=DEV)[:, None]

    def stencil(self, t):
        """(cell index [n], weight [n]) of every corner of the shape function."""
        axes = []
        for a in range(3):
            if self.n[a] == 1:
                axes.append([(torch.zeros_like(self.pos[a], dtype=torch.int64), torch.ones_like(self.pos[a]))])
                continue
            u = (self.pos[a] + self.v[a] * t) / self.dx[a] - 0.5
            if self.shape == 1:
                first = torch.floor(u)
                x = u - first
                ws = (1.0 - x, x)
            else:
                near = torch.floor(u + 0.5)
                x = u - near
                first = near - 1.0
                ws = (0.5 * (0.5 - x) ** 2, 0.75 - x * x, 0.5 * (0.5 + x) ** 2)
            axes.append([(torch.remainder(first.to(torch.int64) + q, self.n[a]), wq) for q, wq in enumerate(ws)])
        return [((cz * self.n[1] + cy) * self.n[0] + cx, wx * wy * wz)
                for cz, wz in axes[2] for cy, wy in axes[1] for cx, wx in axes[0]]

    def grid(self, st, x):
        """Deposit x [9][n] as density and flux: [4][9][cells]."""
        cells = self.n[0] * self.n[1] * self.n[2]
        rows = []
        for g in range(4):
            src = x if g == 0 else x * self.v[g - 1]
            out = torch.zeros((9, cells), dtype=torch.float64, device=DEV)
            for idx, w in st:
                out = out.index_add_(1, idx, src * w)
            rows.append(out)
        return rows

    def source(self, y):
        return self.wN * y[:9] - self.wNb * (y[9:] * self.sign)

    def slope(self, t, y):
        st = self.stencil(t)
        G = self.grid(st, self.source(y))
        hnn = 0.0
        for idx, w in st:
            m = G[0][:, idx]
            for a in range(3):
                m = m - self.v[a] * G[1 + a][:, idx]
            hnn = hnn + w * m
        h = self.hvac + self.vmat + hnn
        hb = (self.hvac - self.vmat - hnn) * self.sign
        return torch.cat([_bracket(h, y[:9]), _bracket(hb, y[9:])])

    def step(self, y, n):
        t, dt = n * self.dt, self.dt
        k1 = self.slope(t, y)
        k2 = self.slope(t + 0.5 * dt, y + 0.5 * dt * k1)
        s = k1 + 2.0 * k2
        k3 = self.slope(t + 0.5 * dt, y + 0.5 * dt * k2)
        s = s + 2.0 * k3
        return y + dt / 6.0 * (s + self.slope(t + dt, y + dt * k3))


def _plain_box(w, wN=None, wNb=None):
    """The particles of a lattice box, direction outer, cell inner."""
    nc, nd = w.ncell_total, w.ndir
    c = torch.arange(nc, device=DEV)
    nx, ny, _ = w.ncell
    home = torch.stack([c % nx, (c // nx) % ny, c // (nx * ny)]).to(torch.float64) + 0.5
    home *= torch.tensor(w.dx, dtype=torch.float64, device=DEV)[:, None]
    if wN is None:
        N, Nb = w.weights()
        wN, wNb = (torch.from_numpy(a / w.dV).to(DEV) for a in (N, Nb))
    each = lambda a: a[:, None].expand(nd, nc).reshape(-1)  # noqa: E731
    v = torch.from_numpy(w.dirs()).to(DEV)
    return _Plain(w.ncell, w.dx, home[:, None, :].expand(3, nd, nc).reshape(3, -1),
                  torch.stack([each(v[:, a]) for a in range(3)]), each(wN), each(wNb), w.hvac(), w.vmat,
                  w.dt, w.shape_order)


def _exact_adjoint(case, seed):
    w = _workload(case, seed)
    p = _adjoint_params(w).requires_grad_(True)
    s = _adjoint_seeds(w, seed).requires_grad_(True)
    mu = torch.from_numpy(w.dirs() @ np.asarray(w.nhat) / np.linalg.norm(w.nhat)).to(DEV)
    wN = (1.0 + 3.0 * p[1] * mu) / w.ndir
    wNb = p[0] * (1.0 + 3.0 * p[2] * mu) / w.ndir
    zero = torch.zeros_like(s[0])
    rows = []
    for o in (0, 4):
        e, t = s[o] ** 2 + s[o + 1] ** 2, s[o + 2] ** 2 + s[o + 3] ** 2
        rows += [1.0 - e - t, e, t, s[o], s[o + 1], s[o + 2], s[o + 3], zero, zero]
    y = torch.stack(rows).reshape(18, -1)

    def one(y, wN, wNb, n):
        return _plain_box(w, wN, wNb).step(y, n)

    for n in range(case["steps"]):
        y = torch.utils.checkpoint.checkpoint(one, y, wN, wNb, n, use_reentrant=False)
    y = y.reshape(18, w.ndir, w.ncell_total)
    nu = (wN[:, None] * (y[1] + y[2])).sum() / (wN.sum() * w.ncell_total)
    nubar = (wNb[:, None] * (y[10] + y[11])).sum() / (wNb.sum() * w.ncell_total)
    (nu + 0.5 * nubar).backward()
    return dict(nu=nu.detach(), nubar=nubar.detach(), params=p.grad, seeds=s.grad)


def _exact_diagnostics(w, box, y, n):
    st = box.stencil(n * w.dt)
    m = torch.cat(box.grid(st, box.wN * y[:9]) + box.grid(st, box.wNb * y[9:]))
    out = {}
    for name, r in (("n", 0), ("fx", 9), ("nbar", 36), ("fxbar", 45)):
        a = np.zeros((3, 3))
        for k in range(3):
            a[k, k] = float(m[r + k].abs().mean())
        for q, (i, j) in enumerate(UP):
            a[i, j] = float(torch.hypot(m[r + 3 + 2 * q], m[r + 4 + 2 * q]).mean())
        out[name] = a
    totals = torch.stack([(box.wN * w.dV * y[:9]).sum(1), (box.wNb * w.dV * y[9:]).sum(1)])
    return dict(moments=m, averages=out, totals=totals.cpu().numpy(), trace=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "adjoint":
        return _exact_adjoint(case, seed)
    with torch.no_grad():
        if kind == "particles":
            w = _particles(case, seed)
            pos, v, N, Nb, y = _particle_arrays(case, w, seed)
            box = _Plain(w.ncell, w.dx, pos.t().contiguous(), v.t().contiguous(), N / w.dV, Nb / w.dV,
                         w.hvac(), w.vmat, w.dt, w.shape_order)
            for n in range(case["steps"]):
                y = box.step(y, n)
            return y
        if kind == "batch":
            out = []
            for i, w in enumerate(_batch_boxes(case, seed)):
                y, box = _state(case, w.nparticles, seed, i), _plain_box(w)
                for n in range(case["steps"]):
                    y = box.step(y, n)
                out.append(y.reshape(18, w.ndir, w.ncell_total))
            return out
        w = _workload(case, seed)
        y, box = _state(case, w.nparticles, seed), _plain_box(w)
        for n in range(case["steps"]):
            y = box.step(y, n)
        if case["output"] == "diagnostics":
            return _exact_diagnostics(w, box, y, case["steps"])
        return y.reshape(18, w.ndir, w.ncell_total)
