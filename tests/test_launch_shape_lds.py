"""dirs_per_wave given and waves left open: 8 waves only where the kernels' LDS
holds their per-direction data, 4 otherwise."""
import numpy as np
import pytest

from oracle import Problem

from test_gpu_steps_1d import box, state
from test_launch_shape_cpu import nbytes

LDS = 160 * 1024


def lds(waves, dpw, shape):
    """LDS bytes of a stage 3 that forms both earlier slopes again, and of an
    adjoint kernel."""
    ne = 3 if shape == 2 else 1
    cells = 64 + 2 * shape + 2
    slot = max(36 * cells, 36 * 64 + waves * 36 * ne)
    dirs = waves * dpw * (9 * ne + 3)
    return 8 * max(slot + dirs + 2 * 36 * (cells + 2), 2 * slot + dirs)


@pytest.mark.parametrize("shape", [1, 2])
@pytest.mark.parametrize("dpw", [16, 32, 48, 49, 50, 51, 52, 64, 96, 120, 128, 150, 200, 256])
def test_waves_fit_the_lds(shape, dpw):
    nz, ndir = 64, 8 * 256
    got = nbytes(nz, ndir, shape, dict(dirs_per_wave=dpw))
    if lds(8, dpw, shape) > LDS:
        assert got == nbytes(nz, ndir, shape, dict(waves=4, dirs_per_wave=dpw))
    else:
        assert got == nbytes(nz, ndir, shape, dict(waves=8, dirs_per_wave=dpw))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,dpw", [(2, 50), (2, 64), (1, 110), (1, 128)])
def test_step_and_adjoint(shape, dpw):
    from paper_2101_02745_amd.sim import Sim
    w = box(70, 260, shape)
    st = state(w)
    sim = Sim.from_workload(w, tuning=dict(dirs_per_wave=dpw))
    sim.set_state(st)
    sim.adjoint_forward(2, 2)
    ref = Problem.from_workload(w).step(st, 2)
    got = sim.get_state().cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
    g, dN, dNb = sim.adjoint_backward(st)
    want = Sim.from_workload(w)
    want.set_state(st)
    want.adjoint_forward(2, 2)
    h, hN, hNb = want.adjoint_backward(st)
    for a, b in ((g.cpu().numpy(), h.cpu().numpy()), (dN, hN), (dNb, hNb)):
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
