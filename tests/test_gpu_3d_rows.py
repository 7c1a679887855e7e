"""The separate 3D kernels read and write the particles with the streaming
cache policy where a row is one wave and whole 128-byte lines, with the
default policy elsewhere, and hand the segments of long rows to the XCDs in
runs: rows on both sides of each line, and work items that the XCDs do not
divide evenly, against the CPU reference at the 1e-12 normwise tolerance of
the other parity tests."""
import pytest

from oracle import Problem
from paper_2101_02745_amd import inputs as I

from test_gpu_parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape_order", [1, 2])
@pytest.mark.parametrize("ncell", [(15, 3, 3), (16, 2, 5), (17, 5, 1), (48, 1, 1), (63, 3, 1),
                                   (64, 2, 2), (65, 1, 1), (129, 5, 3)])
def test_rows(ncell, shape_order):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2101_02745_amd.sim import Sim
    w = I.Workload(name="rows", ncell=ncell, length=tuple(0.5 * n for n in ncell), ndir=26, dt=0.1,
                   steps=0, f=0.1, fbar=-0.2, nbar_over_n=1.2, seed=5, alpha=0.05,
                   shape_order=shape_order)
    s0 = w.state0()
    sim = Sim.from_workload(w, tuning={"fused": 2})
    sim.set_state(s0)
    sim.step(4)
    ref = Problem.from_workload(w).step(s0, 4)
    assert_parity(sim.get_state().cpu().numpy(), ref, what=f"{ncell} shape {shape_order}")


@pytest.mark.parametrize("ncell,ndir,shape_order", [
    ((65, 40, 32), 6, 1),    # 2560 row segments: the last with four waves a row
    ((65, 43, 31), 6, 1),    # 2666: one wave a row, ragged patches
    ((65, 61, 31), 3, 2),    # 3782: four waves, one without a direction
    ((65, 62, 31), 3, 2),    # 3844: one
])
def test_waves_per_deposit_row(ncell, ndir, shape_order):
    """The deposits split a row's directions over four waves in boxes with few
    rows: both sides of the line, both shapes, state and moments."""
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2101_02745_amd.sim import Sim
    w = I.Workload(name="rows", ncell=ncell, length=tuple(0.5 * n for n in ncell), ndir=ndir, dt=0.1,
                   steps=0, f=0.1, fbar=-0.2, nbar_over_n=1.2, seed=5, alpha=0.05,
                   shape_order=shape_order)
    s0 = w.state0()
    P = Problem.from_workload(w)
    sim = Sim.from_workload(w)
    sim.set_state(s0)
    sim.step(2)
    ref = P.step(s0, 2)
    assert_parity(sim.get_state().cpu().numpy(), ref, what=f"{ncell} shape {shape_order}")
    m, mref = sim.moments().cpu().numpy(), P.moments(ref, 2 * w.dt)
    assert np.abs(m - mref.reshape(m.shape)).max() <= 1e-12 * np.abs(mref).max()
