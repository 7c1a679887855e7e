"""The built-in 1D launch shape on the CPU: no box asks for more workspace
than with 4 waves in about 1024 workgroups (the shape the fixed scratch of
fpic_step_noalloc is sized with)."""
import ctypes as C

import numpy as np
import pytest

from paper_2101_02745_amd import _lib
from paper_2101_02745_amd import inputs as I
from paper_2101_02745_amd._lib import HostConfig


def nbytes(nz, ndir, shape, tune):
    dirs = np.tile(I.golden_antipodal_directions(6), (ndir // 6 + 1, 1))[:ndir]
    w = np.full(ndir, 1.0 / ndir)
    cfg = HostConfig((1, 1, nz), (1.0, 1.0, 1.0), dirs, w, w, np.zeros((3, 3)), 0.1, shape)
    n = C.c_size_t()
    t = _lib.tuning(tune)
    _lib.check(_lib.load().fpic_workspace_bytes(C.byref(cfg.c), C.byref(t) if t else None, C.byref(n)))
    return n.value


@pytest.mark.parametrize("shape", [1, 2])
@pytest.mark.parametrize("nz,ndir", [(1, 1), (1, 165000), (1, 60000), (2, 80001), (65, 2530), (64, 2600),
                                     (63, 129), (129, 1281), (700, 235), (2048, 80), (20000, 8),
                                     (160000, 1), (2048, 378), (30000, 92)])
def test_no_more_workspace(nz, ndir, shape):
    wavedirs = -(-nz // 64) * ndir
    dpw = max(1, min(64, -(-wavedirs // 4096)))
    assert nbytes(nz, ndir, shape, None) <= nbytes(nz, ndir, shape, dict(waves=4, dirs_per_wave=dpw))
