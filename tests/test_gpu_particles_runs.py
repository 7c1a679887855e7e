"""The stage kernels deposit a workgroup's 256 particles run by run (a run:
the particles with the same first cell), by one of three routes that the
particles' spread chooses: box accumulators in LDS, a box whose cells do not
fit them (straight to the grid, still run by run), or cells too far apart to
sort (straight to the grid, particle by particle).  Each route against the CPU
reference at the 1e-12 normwise tolerance of the other parity tests, and, for
the exact sums, bit for bit under another order of the same particles."""
import numpy as np
import pytest

from oracle import ParticleProblem
from paper_2101_02745_amd import inputs as I

from test_gpu_parity import assert_parity

pytestmark = pytest.mark.gpu

# ncell, particles per cell, shape order, every which particle is kept
CASES = [
    ((1, 1, 3), 171, 1, 1),      # runs of 171: several waves share one, ragged last workgroup
    ((1, 1, 16), 16, 2, 1),      # exactly one workgroup
    ((1, 1, 257), 1, 1, 1),      # runs of one, one particle in the last workgroup
    ((1, 1, 3000), 1, 2, 11),    # box cells beyond the slot map, first cells sorted
    ((1, 1, 9000), 1, 1, 29),    # first cells too far apart
    ((6, 5, 4), 40, 1, 1),       # accumulators in LDS
    ((12, 10, 8), 3, 1, 1),      # more cells than accumulators
    ((6, 5, 4), 40, 2, 1),       # the same, from the wider stencil
    ((64, 64, 3), 1, 1, 1),      # workgroups across two planes: too far apart
    ((40, 1, 30), 2, 2, 1),      # a flat box
    ((2, 3, 1), 33, 1, 1),       # stencils that wrap onto themselves
]


@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("ncell,ppc,order,every", CASES)
def test_deposit_routes(ncell, ppc, order, every, exact):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2101_02745_amd.particles import ParticleSim
    length = tuple(1.0 if n == 1 else 0.4 * n for n in ncell)
    w = I.ParticleWorkload(name="runs", ncell=ncell, length=length, ppc=ppc, ndir=26, dt=0.1, steps=0,
                           f=0.1, fbar=-0.3, nbar_over_n=0.9, alpha=1e-3, shape_order=order, seed=7)
    keep = np.arange(0, w.nparticles, every)
    pos, dirs, st = w.positions()[keep], w.dirs()[keep], w.state0()[:, keep]
    N, Nb = (a[keep] * every for a in w.weights())
    P = ParticleProblem(ncell, w.dx, pos, dirs, N, Nb, w.hvac(), w.dt, shape_order=order)
    ref = P.step(st, 5)

    def gpu(perm):
        sim = ParticleSim(ncell, w.dx, keep.size, w.hvac(), w.dt, order, sort_every=2, exact=exact)
        sim.set(pos[perm], dirs[perm], N[perm], Nb[perm], st[:, perm])
        sim.step(5)
        out = np.empty_like(ref)
        out[:, perm] = sim.get_state().cpu().numpy()
        sim.close()
        return out

    got = gpu(np.arange(keep.size))
    assert_parity(got, ref, what=f"{ncell} ppc {ppc} order {order}")
    if exact:
        assert np.array_equal(got, gpu(np.random.RandomState(3).permutation(keep.size)))


@pytest.mark.parametrize("npart", [1, 255, (1 << 18) - 1, 1 << 18, (1 << 18) + 57])
def test_state_in_the_callers_order(npart):
    """get_state undoes the sort, component by component or, from 2^18
    particles on, by whole lines: bit for bit what was set."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2101_02745_amd.particles import ParticleSim
    rng = np.random.RandomState(5)
    pos = rng.random_sample((npart, 3)) * (6.0, 5.0, 4.0)
    dirs = I.directions(26)[np.arange(npart) % 26]
    state = rng.standard_normal((18, npart))
    sim = ParticleSim((6, 5, 4), (1.0, 1.0, 1.0), npart, np.zeros((3, 3), complex), 0.1)
    sim.set(pos, dirs, np.ones(npart), np.ones(npart), state)
    assert np.array_equal(sim.get_state().cpu().numpy(), state)
    sim.close()
