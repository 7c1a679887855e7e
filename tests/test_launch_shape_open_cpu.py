"""The built-in 1D launch shape where the caller gives a part of it, on the
CPU: no box asks for more workspace than with its waves in about 1024
workgroups, so that fpic_step_noalloc's fixed scratch holds the same boxes."""
import pytest

from test_launch_shape_cpu import nbytes

NOALLOC_SCRATCH = 64 << 20


def dirs_per_wave(nz, ndir, waves):
    wavedirs = -(-nz // 64) * ndir
    return max(1, min(64, -(-wavedirs // (1024 * waves))))


@pytest.mark.parametrize("waves", [1, 2, 4, 8])
@pytest.mark.parametrize("shape", [1, 2])
@pytest.mark.parametrize("nz,ndir", [(1, 98787), (1, 100446), (3, 35890), (9, 11757), (41, 1374), (169, 594),
                                     (2319, 8), (64, 2600), (2048, 80), (700, 235), (20000, 8), (4000, 378)])
def test_no_more_workspace(nz, ndir, shape, waves):
    want = nbytes(nz, ndir, shape, dict(waves=waves, dirs_per_wave=dirs_per_wave(nz, ndir, waves)))
    got = nbytes(nz, ndir, shape, dict(waves=waves))
    assert got <= want
    state = 18 * 8 * nz * ndir
    if want - state <= NOALLOC_SCRATCH:
        assert got - state <= NOALLOC_SCRATCH
