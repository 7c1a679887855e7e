"""The stage kernels' deposit where a workgroup's 256 particles are spread out:
too many cells for a slot each (straight to the grid, run by run), and first
cells too far apart to sort (straight to the grid, particle by particle).  Which
of them a case reaches is worked out here from the positions, by the kernels'
rule, and asserted.  Against the CPU reference at the 1e-12 normwise tolerance
of the other parity tests, and, for the exact sums, bit for bit under another
order of the same particles."""
import numpy as np
import pytest

from oracle import ParticleProblem
from paper_2101_02745_amd import inputs as I

from test_gpu_parity import assert_parity

pytestmark = pytest.mark.gpu


def routes(pos, ncell, dx, order):
    """The routes of the workgroups' deposit at the particles' positions, in
    cell order: 'apart', 'grid' or 'box' (a box of cells that may have slots)."""
    n, sw = np.array(ncell), order + 1
    u = pos / dx - 0.5
    low = np.floor(u)
    key = np.where(n > 1, low, 0).astype(int) % n
    first = low + (u - low >= 0.5) - 1 if order == 2 else low
    first = np.where(n > 1, first, 0).astype(int) % n
    sort = np.argsort((key[:, 2] * n[1] + key[:, 1]) * n[0] + key[:, 0], kind="stable")
    d3 = ncell[0] * ncell[1] > 1
    out = []
    for b in range(0, len(pos), 256):
        f = first[sort[b:b + 256]]
        o = f - f[0]
        o = np.where(2 * o > n, o - n, np.where(2 * o <= -n, o + n, o))
        ext = o.max(0) - o.min(0) + 1
        if not d3:
            ext[:2] = 1
        cells = np.prod(ext + (sw - 1) * (np.arange(3) >= (0 if d3 else 2)))
        out.append("apart" if np.prod(ext) > 4096 or max(ext[1:]) > 1024 else "grid" if cells > 1024 else "box")
    return out


def every(ncell, k):
    """One particle in every k-th cell."""
    c = np.arange(0, ncell[0] * ncell[1] * ncell[2], k)
    home = np.stack((c % ncell[0], c // ncell[0] % ncell[1], c // (ncell[0] * ncell[1])), axis=1)
    return home + np.random.RandomState(k).random_sample(home.shape)


def spans(nz, span):
    """Groups of 256 particles in a 1D box, each spread evenly over span cells
    (the first cells of both ends included), near the cells' centres."""
    starts = np.arange(0, nz - span, span)
    z = (starts[:, None] + np.round(np.arange(256) * (span - 1) / 255)).ravel() + 0.6
    return np.stack((np.full(z.size, 0.5), np.full(z.size, 0.5), z), axis=1)


# route, ncell, shape order, positions in cells
CASES = [
    ("apart", (40, 40, 40), 1, every((40, 40, 40), 23)),
    ("apart", (40, 40, 40), 2, every((40, 40, 40), 23)),
    ("apart", (5000, 2, 1), 1, every((5000, 2, 1), 19)),      # more than 4096 cells in x alone
    ("apart", (1, 1, 9000), 2, every((1, 1, 9000), 29)),
    ("apart", (1, 1, 9000), 1, spans(9000, 1025)),            # one cell too many for the packed index
    ("grid", (16, 16, 16), 1, every((16, 16, 16), 10)),
    ("grid", (16, 16, 16), 2, every((16, 16, 16), 10)),
    ("grid", (3000, 1, 1), 1, every((3000, 1, 1), 9)),
    ("grid", (1, 1, 9000), 1, spans(9000, 1024)),             # the most that are sorted in a 1D box
    ("grid", (1, 1, 9000), 2, spans(9000, 1024)),
]


@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_spread(case, exact):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2101_02745_amd.particles import ParticleSim
    route, ncell, order, pos = CASES[case]
    dx = np.full(3, 0.4)
    dx[[n == 1 for n in ncell]] = 1.0
    assert route in routes(pos * dx, ncell, dx, order)
    w = I.ParticleWorkload(name="spread", ncell=ncell, length=tuple(dx * ncell), ppc=1, ndir=26, dt=0.1, steps=0,
                           f=0.1, fbar=-0.3, nbar_over_n=0.9, alpha=1e-3, shape_order=order, seed=7)
    n, scale = len(pos), np.prod(ncell) / len(pos)
    dirs, st = w.dirs()[:n], w.state0()[:, :n]
    N, Nb = (a[:n] * scale for a in w.weights())
    P = ParticleProblem(ncell, dx, pos * dx, dirs, N, Nb, w.hvac(), w.dt, shape_order=order)
    ref = P.step(st, 5)
    mref = P.moments(ref, 5 * w.dt)

    def gpu(perm):
        sim = ParticleSim(ncell, dx, n, w.hvac(), w.dt, order, sort_every=2, exact=exact)
        sim.set((pos * dx)[perm], dirs[perm], N[perm], Nb[perm], st[:, perm])
        sim.step(5)
        out = np.empty_like(ref)
        out[:, perm] = sim.get_state().cpu().numpy()
        mom = sim.moments().cpu().numpy()
        assert np.array_equal(mom, sim.moments().cpu().numpy()) or not exact
        sim.step(1)     # the sums of the next stages start from zero again
        last = np.empty_like(ref)
        last[:, perm] = sim.get_state().cpu().numpy()
        sim.close()
        return out, mom, last

    got, mom, last = gpu(np.arange(n))
    assert_parity(got, ref, what=f"{route} {ncell} order {order}")
    assert np.abs(mom - mref.reshape(mom.shape)).max() <= 1e-12 * np.abs(mref).max()
    assert_parity(last, P.step(ref, 1, 5), what=f"{route} {ncell} order {order}, step after the moments")
    if exact:
        for a, b in zip((got, mom, last), gpu(np.random.RandomState(3).permutation(n))):
            assert np.array_equal(a, b)
