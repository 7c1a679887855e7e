"""Whole 1D steps in one launch (small boxes in their built-in shape) against
one launch per stage: the same bits after several calls, for tiles of every
kind (one tile, ragged, a last tile of one cell, wrapped columns), both
shapes, batches, launches that follow one another, and boxes just outside the
rule; and the same bits where a launch's workgroups do not run together."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2101_02745_amd import _lib
from paper_2101_02745_amd import inputs as I
from paper_2101_02745_amd._lib import HostConfig
from paper_2101_02745_amd.sim import Batch, Sim

pytestmark = pytest.mark.gpu


def box(nz, ndir, shape, dz=0.098, dt=0.1):
    return I.Workload(name="t", ncell=(1, 1, nz), length=(1.0, 1.0, nz * dz), ndir=ndir, dt=dt, steps=1,
                      nbar_over_n=0.9, f=0.1, fbar=-0.2, nhat=(0.3, 0.2, 0.9), vmat=(0.4, 0.1, 0.0),
                      shape_order=shape, seed=nz + ndir)


def state(w):
    r = np.random.RandomState(w.seed)
    s = np.zeros((18, w.ndir, w.ncell_total))
    for o in (0, 9):
        p = r.normal(size=(3, 2) + s.shape[1:])
        p /= np.sqrt((p ** 2).sum((0, 1)))
        z = p[:, 0] + 1j * p[:, 1]
        for k in range(3):
            s[o + k] = np.abs(z[k]) ** 2
        for q, (a, b) in enumerate(((0, 1), (0, 2), (1, 2))):
            m = z[a] * z[b].conj()
            s[o + 3 + 2 * q], s[o + 4 + 2 * q] = m.real, m.imag
    return s


@pytest.mark.parametrize("shape", [1, 2])
@pytest.mark.parametrize("nz,ndir", [(15, 8), (16, 8), (17, 26), (63, 10), (64, 24), (65, 24), (66, 26), (67, 6),
                                     (128, 92), (129, 26), (200, 92), (777, 92), (2048, 64), (2049, 64),
                                     (100, 192), (100, 194)])
def test_same_bits(nz, ndir, shape):
    w = box(nz, ndir, shape)
    st = state(w)
    sims = [Sim.from_workload(w), Sim.from_workload(w, tuning=dict(fused=2))]
    for s in sims:
        s.set_state(st, 37)
        for n in (1, 3, 9):
            s.step(n)
    assert sims[0].step_index() == sims[1].step_index() == 37 + 13
    assert torch.equal(sims[0].get_state(), sims[1].get_state())
    assert torch.equal(sims[0].moments(), sims[1].moments())


@pytest.mark.parametrize("nz,ndir,shape", [(16, 8, 1), (65, 26, 2), (200, 24, 1)])
def test_workgroups_not_together(nz, ndir, shape):
    """With no wait for the other workgroups, one of them runs every step."""
    w = box(nz, ndir, shape)
    st = state(w)
    sims = [Sim.from_workload(w), Sim.from_workload(w, tuning=dict(fused=2))]
    f = getattr(_lib.load(), "_ZN4fpic16set_arrive_ticksEPvy")
    f.argtypes = [C.c_void_p, C.c_uint64]
    for s in sims:
        s.set_state(st, 3)
    for ticks, n in ((0, 2), (10 ** 8, 3), (0, 1), (10 ** 8, 2)):
        assert f(sims[0].ctx, ticks) == 0
        for s in sims:
            s.step(n)
    assert sims[0].step_index() == sims[1].step_index() == 11
    assert torch.equal(sims[0].get_state(), sims[1].get_state())
    assert torch.equal(sims[0].moments(), sims[1].moments())


def test_batch_same_bits():
    ws = [box(40, 24, 1), box(65, 26, 1, dz=0.2), box(130, 64, 1, dz=0.15, dt=0.05)]
    bs = [Batch([HostConfig.from_workload(w) for w in ws], tuning=t) for t in (None, dict(fused=2))]
    for b in bs:
        for i, w in enumerate(ws):
            b.set_state(i, state(w), 5 * i)
        b.step(2)
        b.step(6)
    for i in range(len(ws)):
        assert torch.equal(bs[0].get_state(i), bs[1].get_state(i))


def test_many_contexts_and_streams():
    """Contexts stepped in turn on streams of their own, no waits between."""
    ws = [box(70 + 5 * i, 24, 1 + i % 2) for i in range(4)]
    streams = [torch.cuda.Stream() for _ in ws]
    sims = []
    for w, q in zip(ws, streams):
        with torch.cuda.stream(q):
            s = Sim.from_workload(w)
            s.set_state(state(w))
            sims.append(s)
    for _ in range(5):
        for s in sims:
            s.step(2)
    for w, s in zip(ws, sims):
        s.sync()
        r = Sim.from_workload(w, tuning=dict(fused=2))
        r.set_state(state(w))
        r.step(10)
        torch.cuda.synchronize()
        assert torch.equal(s.get_state(), r.get_state())
