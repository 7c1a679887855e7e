"""get_state of a large box (by whole lines, with a scratch array in between)
touches nothing that the steps go on with, also where it is replayed from a
captured graph after a sort has moved the particles to the other set."""
import numpy as np
import pytest
import torch

from paper_2101_02745_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ppc,shape", [(86, 1), (90, 2)])
def test_replayed_after_a_sort(ppc, shape):
    from paper_2101_02745_amd.particles import ParticleSim
    ncell = (1, 1, 3072)        # 264,192 and 276,480 particles
    w = I.ParticleWorkload(name="g", ncell=ncell, length=(1.0, 1.0, 0.4 * 3072), ppc=ppc, ndir=26, dt=0.1, steps=0,
                           f=0.1, fbar=-0.3, nbar_over_n=0.9, alpha=1e-3, shape_order=shape, seed=7)
    N, Nb = w.weights()
    q = torch.cuda.Stream()
    out = []
    with torch.cuda.stream(q):
        for replay in (False, True):
            sim = ParticleSim(ncell, w.dx, w.nparticles, w.hvac(), w.dt, shape, sort_every=2)
            sim.set(w.positions(), w.dirs(), N, Nb, w.state0())
            sim.sync()
            if replay:
                g = torch.cuda.CUDAGraph()
                with torch.cuda.graph(g, stream=q):
                    first = sim.get_state()
                g.replay()
                q.synchronize()
                assert np.array_equal(first.cpu().numpy(), w.state0())
            sim.step(2)
            if replay:
                g.replay()
                q.synchronize()
            sim.step(3)
            sim.sync()
            out.append(sim.get_state().cpu().numpy())
            sim.close()
    assert np.array_equal(out[0], out[1])
