"""How many waves share a destination row in the 3D deposits follows the rows,
the directions and the components: both sides of each line, both shapes, state
and moments, against the CPU reference at the 1e-12 normwise tolerance of the
other parity tests."""
import numpy as np
import pytest

from oracle import Problem
from paper_2101_02745_amd import inputs as I

from test_gpu_parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncell,ndir,shape_order", [
    ((5, 32, 16), 2, 1),     # 512 rows: four waves, two without a direction
    ((5, 19, 27), 6, 1),     # 513: one, below 8 directions
    ((5, 19, 27), 8, 1),     # four
    ((4, 32, 24), 6, 2),     # 768: four (moments one)
    ((4, 769, 1), 6, 2),     # 769: one
    ((3, 97, 19), 8, 1),     # 1843: four
    ((3, 97, 19), 8, 2),
    ((3, 61, 31), 8, 1),     # 1891: one, as the rows fill the chip once
    ((3, 32, 64), 8, 1),     # 2048: one
    ((3, 683, 3), 8, 1),     # 2049: four
    ((3, 683, 3), 8, 2),     # four, the moments too
    ((65, 40, 32), 8, 1),    # 2560 row segments: the last with four
    ((65, 40, 32), 8, 2),    # the moments' last with four
    ((65, 43, 31), 8, 2),    # 2666: moments one
    ((65, 61, 31), 8, 2),    # 3782: four
    ((65, 62, 31), 8, 2),    # 3844: one
])
def test_waves_per_deposit_row(ncell, ndir, shape_order):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2101_02745_amd.sim import Sim
    w = I.Workload(name="rows", ncell=ncell, length=tuple(0.5 * n for n in ncell), ndir=ndir, dt=0.1,
                   steps=0, f=0.1, fbar=-0.2, nbar_over_n=1.2, seed=5, alpha=0.05,
                   shape_order=shape_order)
    s0 = w.state0()
    P = Problem.from_workload(w)
    sim = Sim.from_workload(w, tuning=dict(fused=2))
    sim.set_state(s0)
    sim.step(2)
    ref = P.step(s0, 2)
    assert_parity(sim.get_state().cpu().numpy(), ref, what=f"{ncell} x {ndir} shape {shape_order}")
    m, mref = sim.moments().cpu().numpy(), P.moments(ref, 2 * w.dt)
    assert np.abs(m - mref.reshape(m.shape)).max() <= 1e-12 * np.abs(mref).max()
