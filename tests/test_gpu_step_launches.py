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
    f.argtypes = [C.c_void_p, C.c_void_p, C.c_uint64, C.c_uint32]
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


def independent_streams():
    """Two streams, the second of which goes on while the first is busy (the
    runtime maps streams to a few hardware queues)."""
    a, x = torch.cuda.Stream(), torch.zeros(1, device="cuda")
    for b in [torch.cuda.Stream() for _ in range(8)]:
        torch.cuda.synchronize()
        with torch.cuda.stream(a):
            torch.cuda._sleep(200_000_000)
            busy = torch.cuda.Event()
            busy.record()
        with torch.cuda.stream(b):
            x.add_(1)
        b.synchronize()
        if not busy.query():
            return a, b
    pytest.skip("no two streams that run side by side")


@pytest.mark.parametrize("nz,ndir", [(32, 26), (200, 92), (2048, 64)])
def test_streams_do_not_wait_for_one_another(nz, ndir):
    """A box whose stream waits behind other work holds up no box on another
    stream, whether both fit the chip together (32 x 26: 4 workgroups, 200 x
    92: 48) or not (2048 x 64: 256)."""
    a, b = independent_streams()
    w = box(nz, ndir, 1)
    sims = []
    for q in (a, b):
        with torch.cuda.stream(q):
            sims.append(Sim.from_workload(w))
            sims[-1].set_state(state(w))
    for s in sims:
        s.step(1)
        s.sync()
    with torch.cuda.stream(a):
        torch.cuda._sleep(2_000_000_000)
        sims[0].step(3)
        sims[0].step(3)
        busy = torch.cuda.Event()
        busy.record()
    sims[1].step(3)
    sims[1].step(3)
    sims[1].sync()
    assert not busy.query()
    sims[0].sync()
    sims[1].step(2)
    sims[0].step(2)
    ref = reference(w, 9)
    for s in sims:
        s.sync()
        assert torch.equal(s.get_state(), ref)
        torch.cuda.synchronize()


def test_adjoint_beside_another_stream():
    """The recomputation of a segment beside a launch that takes the whole
    chip: gradients bit for bit those of a context alone."""
    a, b = independent_streams()
    w, wide = box(130, 24, 1), box(2048, 64, 1)
    g = torch.from_numpy(state(w)).cuda()

    def gradients(q):
        with torch.cuda.stream(q):
            s = Sim.from_workload(w)
            s.set_state(state(w))
            s.adjoint_forward(5, 2)
            return s.adjoint_backward(g)

    torch.cuda.synchronize()
    alone = gradients(b)
    with torch.cuda.stream(a):
        s = Sim.from_workload(wide)
        s.set_state(state(wide))
        torch.cuda._sleep(1_000_000_000)
        s.step(2)
    beside = gradients(b)
    torch.cuda.synchronize()
    assert torch.equal(alone[0], beside[0])
    assert (alone[1] == beside[1]).all() and (alone[2] == beside[2]).all()


# waits, in ticks of 10 ns, from none to about that of all workgroups of a
# launch for one another: teams of few workgroups and of many
WAITS = (0, 40, 80, 120, 160, 240, 10 ** 8)


@pytest.mark.parametrize("nz,ndir,shape", [(2048, 64, 1), (777, 92, 2), (200, 92, 1), (16, 26, 2)])
def test_teams(nz, ndir, shape):
    """Where a launch's workgroups are not resident together in time, those
    that are share the work: the same bits, launch after launch."""
    w = box(nz, ndir, shape)
    s = Sim.from_workload(w)
    s.set_state(state(w), 3)
    for ticks in WAITS:
        set_waits(s, ticks, 2 * 10 ** 9)
        s.step(2)
    s.sync()
    assert s.step_index() == 3 + 2 * len(WAITS)
    assert torch.equal(s.get_state(), reference(w, 2 * len(WAITS), 3))


def test_teams_in_a_batch():
    """Boxes of other sizes and start steps, several of one workgroup."""
    ws = [box(40, 24, 1), box(65, 26, 1, dz=0.2), box(130, 64, 1, dz=0.15, dt=0.05), box(16, 10, 1)]
    b = Batch([HostConfig.from_workload(w) for w in ws])
    for i, w in enumerate(ws):
        b.set_state(i, state(w), 5 * i)
    for ticks in WAITS:
        set_waits(b, ticks, 2 * 10 ** 9)
        b.step(3)
    b.sync()
    for i, w in enumerate(ws):
        assert torch.equal(b.get_state(i), reference(w, 3 * len(WAITS), 5 * i))


@pytest.mark.parametrize("nz,ndir,shape", [(130, 24, 1), (65, 26, 2), (512, 128, 1)])
def test_teams_in_the_adjoint(nz, ndir, shape):
    """The recomputation keeps every stage's grids and slopes for the reverse
    sweep: the gradients of a team are those of the whole launch."""
    w = box(nz, ndir, shape)
    g = torch.from_numpy(state(w)).cuda()

    def gradients(ticks):
        s = Sim.from_workload(w)
        s.set_state(state(w), 2)
        s.adjoint_forward(5, 2)
        if ticks is not None:
            set_waits(s, ticks, 2 * 10 ** 9)
        return s.adjoint_backward(g)

    want = gradients(None)
    for ticks in WAITS:
        got = gradients(ticks)
        assert torch.equal(got[0], want[0])
        assert (got[1] == want[1]).all() and (got[2] == want[2]).all()


def launches(s):
    """Launches of whole steps so far, -1 for a context that makes none."""
    f = _lib.load().fpic_test_step_launches
    f.argtypes = [C.c_void_p, C.c_void_p]
    return f(getattr(s, "ctx", None), getattr(s, "b", None))


@pytest.mark.parametrize("nz,ndir,shape,whole", [(15, 8, 1, False), (16, 8, 2, True), (32, 26, 1, True),
                                                 (777, 92, 2, True), (2048, 64, 1, True), (2049, 64, 1, False),
                                                 (100, 192, 1, True), (100, 194, 1, False)])
def test_which_boxes_take_whole_steps(nz, ndir, shape, whole):
    """Both sides of the rule: at least 16 cells, at most 256 workgroups and 24
    direction groups, one direction a wave, every slope stored by choice."""
    w = box(nz, ndir, shape)
    s = Sim.from_workload(w)
    s.set_state(state(w))
    s.step(3)
    s.step(600)
    assert launches(s) == (3 if whole else -1)    # 3, 512 and 88 steps
    for tune in (dict(fused=2), dict(waves=8, dirs_per_wave=2)):
        assert launches(Sim.from_workload(w, tuning=tune)) == -1


def test_batches_and_the_adjoint_take_whole_steps():
    ws = [box(40, 24, 1), box(65, 26, 1)]
    b = Batch([HostConfig.from_workload(w) for w in ws])
    for i, w in enumerate(ws):
        b.set_state(i, state(w))
    b.step(4)
    assert launches(b) == 1
    w = box(130, 24, 1)
    s = Sim.from_workload(w)
    s.set_state(state(w))
    s.adjoint_forward(5, 2)
    assert launches(s) == 3
    s.adjoint_backward(state(w))
    assert launches(s) == 6


def test_steps_while_the_stream_is_captured():
    """A box that runs whole steps does under capture what one launch per stage
    does, and goes on with whole steps afterwards."""
    w = box(65, 26, 2)
    q = torch.cuda.Stream()
    got = []
    for tune in (None, dict(fused=2)):
        with torch.cuda.stream(q):
            s = Sim.from_workload(w, tuning=tune)
            s.set_state(state(w), 4)
            s.step(1)
            s.sync()
        before = launches(s)
        g = torch.cuda.CUDAGraph()
        x = torch.zeros(4, device="cuda")
        with torch.cuda.graph(g, stream=q):
            x.add_(1.0)
            s.step(11)
        assert launches(s) == before
        for _ in range(3):
            g.replay()
            torch.cuda.synchronize()
        s.step(2)
        s.sync()
        assert launches(s) == (before + 1 if tune is None else -1)
        got.append((s.step_index(), s.get_state()))
        torch.cuda.synchronize()
    assert got[0][0] == got[1][0]
    assert torch.equal(got[0][1], got[1][1])
    assert torch.equal(got[0][1], reference(w, got[0][0] - 4, 4))


@pytest.mark.parametrize("nz,ndir,shape", [(16, 26, 1), (65, 26, 2), (130, 64, 1), (200, 92, 2)])
@pytest.mark.parametrize("step0", [0, 10 ** 9])
def test_fast_particles(nz, ndir, shape, step0):
    """Steps of nearly two cells: most anchors move on in every half step."""
    w = box(nz, ndir, shape, dz=0.0505)
    s = Sim.from_workload(w)
    s.set_state(state(w), step0)
    s.step(7)
    s.step(4)
    s.sync()
    assert launches(s) == 2
    assert torch.equal(s.get_state(), reference(w, 11, step0))


def test_threads():
    """Contexts on streams of their own, stepped by a thread each, together
    larger than the chip: every one as if it were alone."""
    import threading
    ws = [box(2048, 64, 1), box(777, 92, 1), box(2000, 60, 2), box(200, 92, 1), box(32, 26, 1), box(130, 24, 2)]
    sims, errors = [], []
    for w in ws:
        with torch.cuda.stream(torch.cuda.Stream()):
            sims.append(Sim.from_workload(w))
            sims[-1].set_state(state(w))
            sims[-1].sync()

    def work(s, seed):
        try:
            for k in range(40):
                s.step(1 + (k * seed) % 4)
                if k % 7 == seed % 7:
                    s.sync()
            s.sync()
        except Exception as e:          # (an exception in a thread would be lost)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(s, i + 1)) for i, s in enumerate(sims)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for i, (s, w) in enumerate(zip(sims, ws)):
        n = sum(1 + (k * (i + 1)) % 4 for k in range(40))
        got = s.get_state()
        s.sync()
        assert s.step_index() == n
        assert torch.equal(got, reference(w, n))
