"""dirs_per_wave given and waves left open: 4 waves, whose LDS holds twice the
directions of 8."""
import numpy as np
import pytest

from oracle import Problem

from test_gpu_steps_1d import box, state
from test_launch_shape_cpu import nbytes


@pytest.mark.parametrize("shape", [1, 2])
@pytest.mark.parametrize("nz,ndir", [(64, 2048), (200, 92), (2048, 378)])
@pytest.mark.parametrize("dpw", [2, 4, 12, 51, 64, 128, 150, 256])
def test_four_waves(nz, ndir, shape, dpw):
    assert nbytes(nz, ndir, shape, dict(dirs_per_wave=dpw)) == \
        nbytes(nz, ndir, shape, dict(waves=4, dirs_per_wave=dpw))


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
