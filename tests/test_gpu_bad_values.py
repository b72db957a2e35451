"""States with a bad value in one cell (NaN, infinities, a negative density or
depth) on the paths that small lattices take against those that large ones
take: the 1D marches against one launch per step, tiles against the marching
strips and planes (a lattice periodic in its last axis, and the same many times
over).  The same bits, flags and first bad step."""
import dataclasses

import numpy as np
import pytest

from paper_2609_18177_amd import arlbm as A
from gpu_common import gpu_lattice, require_gpu, say
from test_gpu_march_strips import MAKE2, P, R, T, _box, _rows_of
from test_gpu_march1d_grid import _problem
from test_gpu_strips import crop

pytestmark = pytest.mark.gpu

VALUES = (np.nan, np.inf, -np.inf, -5.0)


def _plant(L, cells, at, value, prec):
    """value in the population k = 0 of the first field of the cells `at`."""
    real, stride = (np.float32 if prec == A.F32 else np.float64), (cells + 63) // 64 * 64 + 1088
    blob = bytearray(L.save_state())
    f = np.frombuffer(blob, dtype=real, count=stride, offset=56).copy()
    f[at] = value
    blob[56:56 + f.nbytes] = f.tobytes()
    L.load_state(bytes(blob))


def _same(a, b, reps=None):
    U, V = a.moments(), b.moments()
    if reps is not None:
        U = np.tile(U, reps)
    return repr(a.sync(check=False)) == repr(b.sync(check=False)) and np.array_equal(U, V, equal_nan=True)


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("kind", ["advection", "euler", "swe", "reactive"])
def test_bad_values_in_1d(kind, prec):
    require_gpu()
    for n in (300, 4096):
        for value in VALUES:
            p = _problem(kind, n, T)
            say(f"[bad value {value}] {kind} {n} cells prec={prec}")
            a, b = (gpu_lattice(p, prec) for _ in range(2))
            for L in (a, b):
                _plant(L, n, n // 3, value, prec)
            a.step(40)
            for _ in range(40):
                b.step(1)
            assert _same(a, b), (n, value)
            a.close()
            b.close()


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system,nx,h,k,xbc", [("advection", 250, 128, 10, T), ("euler", 250, 100, 12, T),
                                               ("swe", 250, 128, 18, R), ("reactive", 118, 90, 21, R)])
def test_bad_values_in_2d(system, nx, h, k, xbc, prec):
    require_gpu()
    p = crop(MAKE2[system](), nx, h, bc=(xbc, xbc, P, P), ox=(256 - nx) // 2, oy=60)
    q = dataclasses.replace(p, ny=k * h, y1=p.y0 + k * (p.y1 - p.y0), U0=np.tile(p.U0, (1, k, 1)),
                            bed=None if p.bed is None else np.tile(p.bed, (k, 1)))
    assert _rows_of(p, prec) > 0 and _rows_of(q, prec) == 0
    at = (h // 2) * nx + nx // 3
    for value in VALUES:
        say(f"[bad value {value}] {system} {nx}x{h} prec={prec}")
        a, b = (gpu_lattice(x, prec) for x in (p, q))
        _plant(a, p.cells, at, value, prec)
        _plant(b, q.cells, at + np.arange(k) * h * nx, value, prec)
        a.step(12)
        b.step(12)
        assert _same(a, b, (1, k, 1)), value
        a.close()
        b.close()


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system,nx,ny,h,k", [("euler", 33, 17, 24, 30), ("euler", 70, 37, 64, 4),
                                              ("advection", 33, 17, 40, 55), ("reactive", 33, 17, 24, 30)])
def test_bad_values_in_3d(system, nx, ny, h, k, prec):
    require_gpu()
    p = _box(system, nx, ny, 72, (T, T, P, P, P, P), 0)
    o, dz = (72 - h) // 2, p.z1 / 72
    p = dataclasses.replace(p, nz=h, z1=h * dz, U0=np.ascontiguousarray(p.U0[:, o:o + h]))
    q = dataclasses.replace(p, nz=k * h, z1=k * h * dz, U0=np.tile(p.U0, (1, k, 1, 1)))
    assert _rows_of(p, prec) > 0 and _rows_of(q, prec) == 0
    at = ((h // 2) * ny + ny // 2) * nx + nx // 3
    for value in VALUES[::3]:
        say(f"[bad value {value}] {system} {nx}x{ny}x{h} prec={prec}")
        a, b = (gpu_lattice(x, prec) for x in (p, q))
        _plant(a, p.cells, at, value, prec)
        _plant(b, q.cells, at + np.arange(k) * h * ny * nx, value, prec)
        a.step(6)
        b.step(6)
        assert _same(a, b, (1, k, 1, 1)), value
        a.close()
        b.close()
