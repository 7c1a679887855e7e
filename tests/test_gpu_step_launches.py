"""Launches of whole 1D steps beside other work: contexts made and stepped on
non-blocking streams, against one launch per stage bit for bit."""
import ctypes as C

import pytest
import torch

from paper_2101_02745_amd import _lib
from paper_2101_02745_amd._lib import HostConfig, check
from paper_2101_02745_amd.sim import Sim

from test_gpu_steps_1d import box, state

pytestmark = pytest.mark.gpu


def reference(w, steps, step0=0):
    """State after steps, one launch per stage."""
    r = Sim.from_workload(w, tuning=dict(fused=2))
    r.set_state(state(w), step0)
    r.step(steps)
    r.sync()
    return r.get_state()


def test_counters_clear_before_the_first_launch():
    """A used workspace, a non-blocking stream, and the null stream busy: the
    counters that a launch's workgroups wait on are clear when it starts."""
    lib = _lib.load()
    w = box(200, 24, 1)
    hc = HostConfig.from_workload(w)
    n = C.c_size_t()
    check(lib.fpic_workspace_bytes(C.byref(hc.c), None, C.byref(n)))
    ws = torch.full((n.value,), 0xff, dtype=torch.uint8, device="cuda")
    st, out = torch.from_numpy(state(w)).cuda(), torch.empty(18, 24, 200, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    q = torch.cuda.Stream()
    torch.cuda._sleep(50_000_000)
    ctx = C.c_void_p()
    check(lib.fpic_create(C.byref(hc.c), None, ws.data_ptr(), n.value, q.cuda_stream, C.byref(ctx)))
    check(lib.fpic_set_state(ctx, st.data_ptr(), 0))
    check(lib.fpic_step(ctx, 5))
    check(lib.fpic_get_state(ctx, out.data_ptr()))
    check(lib.fpic_sync(ctx))
    lib.fpic_destroy(ctx)
    assert torch.equal(out, reference(w, 5))
