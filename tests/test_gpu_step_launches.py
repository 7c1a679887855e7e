"""Launches of whole 1D steps beside other work: contexts made and stepped on
non-blocking streams, against one launch per stage bit for bit."""
import ctypes as C

import pytest
import torch

from paper_2101_02745_amd import _lib
from paper_2101_02745_amd._lib import FpicError, HostConfig, check
from paper_2101_02745_amd.sim import Batch, Sim

from test_gpu_steps_1d import box, state

pytestmark = pytest.mark.gpu


def reference(w, steps, step0=0):
    """State after steps, one launch per stage."""
    r = Sim.from_workload(w, tuning=dict(fused=2))
    r.set_state(state(w), step0)
    r.step(steps)
    r.sync()
    return r.get_state()


def set_waits(s, arrive, barrier):
    f = _lib.load().fpic_test_step_waits
    f.argtypes = [C.c_void_p, C.c_void_p, C.c_uint64, C.c_uint64]
    check(f(getattr(s, "ctx", None), getattr(s, "b", None), arrive, barrier))


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


def test_given_up_wait_is_reported():
    """Workgroups that give up a barrier (here at once, instead of after 20 s)
    leave no state that could pass for a result, and every later call of the
    context is an error; other contexts go on."""
    w = box(200, 92, 1)
    s, other = Sim.from_workload(w), Sim.from_workload(w)
    for q in (s, other):
        q.set_state(state(w))
    set_waits(s, 10 ** 8, 0)
    torch.cuda._sleep(100_000_000)
    s.step(3)
    got = s.get_state()           # queued before the launch has run
    torch.cuda.synchronize()
    assert torch.isnan(got).all()
    m = torch.zeros(72, 200, dtype=torch.float64, device="cuda")
    for call in (s.sync, s.get_state, s.moments, s.flavor_totals, s.check, s.step_index, s.step,
                 lambda: s.set_state(state(w)), lambda: s.domain_averages(m), lambda: s.profile(1),
                 lambda: s.adjoint_forward(2)):
        with pytest.raises(FpicError):
            call()
    s.close()
    other.step(3)
    assert torch.equal(other.get_state(), reference(w, 3))


def test_given_up_wait_in_a_batch():
    ws = [box(130, 64, 1), box(65, 26, 1)]
    b = Batch([HostConfig.from_workload(w) for w in ws])
    for i, w in enumerate(ws):
        b.set_state(i, state(w))
    set_waits(b, 10 ** 8, 0)
    torch.cuda._sleep(100_000_000)
    b.step(2)
    got = [b.get_state(i) for i in range(2)]
    torch.cuda.synchronize()
    assert all(torch.isnan(g).all() for g in got)
    for call in (b.sync, b.step, b.flavor_totals, lambda: b.get_state(1), lambda: b.set_state(1, state(ws[1]))):
        with pytest.raises(FpicError):
            call()
