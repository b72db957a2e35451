"""The marching 2D and 3D steps, and the tiles of more than one per CU, at the
shapes where they can go wrong.

Small lattices are stepped in tiles, so the geometry of the marching strips
(one or two columns per lane, ragged last strips, every face, the bed, the
omega export, null steps, the guard against stray writes) and of the marching
planes (ragged tiles in x and y, plane chunks) is checked here on narrow
lattices tall enough to be past the tiles' line, at few cells: FP64 against the
oracle bit for bit (reactive Euler within 1e-12 pointwise), FP32 against it
within a bound and against the batched server's strips bit for bit.  And both
precisions against the tiles bit for bit: a lattice that is periodic in y (z)
and one that holds it many times over, the first in tiles, the second
marching, take the same steps."""
import dataclasses

import numpy as np
import pytest

from paper_2609_18177_amd import arlbm as A
from paper_2609_18177_amd import workloads as W
from gpu_common import fp64_parity_ok, gpu_lattice, oracle_run, rel_l1, require_gpu, say
from test_gpu_strips import SENTINEL, TOL_FP32, TOL_OMEGA32_1, _served, crop
from test_gpu_3d import TOL_FP32 as TOL3_FP32
from test_gpu_tile2d import LARGE, _served_beside

pytestmark = pytest.mark.gpu

T, R, P = A.TRANSMISSIVE, A.REFLECTIVE, A.PERIODIC
MAKE2 = {"advection": lambda: W.advection_sine_2d(n=256, ax=0.8, ay=-0.5), "euler": lambda: W.euler_seeded_2d(4, n=256),
         "swe": lambda: W.swe_bed_2d(1, n=256), "reactive": lambda: W.reactive_seeded_2d(1, n=256)}
TOL3 = {"advection": TOL3_FP32, "euler": TOL3_FP32, "reactive": 2e-3}  # FP32 in 3D, as for the cubes of each system
MAKE3 = {"advection": W.advection_sine_3d, "euler": W.euler_octants_3d, "reactive": W.reactive_sphere_3d}


def _rows_of(p, precision=A.F32):
    """Height of the lattice's tiles, 0 where it marches."""
    return int(A.plan_tiles([A.config_from(p, precision=precision)])[0][0])


def _there_and_back(n, base):
    """n indices that walk 0 .. base-1 and back again: the data stay continuous."""
    i = np.arange(n) % (2 * base)
    return np.where(i < base, i, 2 * base - 1 - i)


def _tall(system, nx, ny, bc, steps):
    """nx columns of the square problem, its rows walked there and back."""
    p = crop(MAKE2[system](), nx, 256, bc=bc, ox=(256 - nx) // 2, steps=steps)
    dx, i = (p.x1 - p.x0) / nx, _there_and_back(ny, 256)
    return dataclasses.replace(p, ny=ny, y0=0.0, y1=ny * dx, U0=np.ascontiguousarray(p.U0[:, i]),
                               bed=None if p.bed is None else np.ascontiguousarray(p.bed[i]))


# widths: fewer columns than a halo is wide, one strip, one column more, odd and
# even, two columns per lane (advection FP32, shallow water) with one strip of
# 120 and two columns more; heights past the tiles' line
CASES2 = [("advection", 4, 5400, (P,) * 4), ("advection", 120, 1900, (T,) * 4), ("advection", 122, 1900, (T, T, P, P)),
          ("advection", 251, 1100, (T,) * 4),
          ("euler", 4, 5400, (R, R, T, T)), ("euler", 58, 5400, (P,) * 4), ("euler", 59, 2700, (R, T, P, P)),
          ("euler", 250, 1090, (T,) * 4), ("euler", 251, 1090, (R,) * 4),
          ("swe", 4, 10300, (T,) * 4), ("swe", 120, 3500, (R,) * 4), ("swe", 122, 3500, (P, P, T, R)),
          ("swe", 249, 2060, (R,) * 4), ("swe", 250, 2060, (P,) * 4),
          ("reactive", 59, 2700, (T, R, R, T)), ("reactive", 250, 1090, (T,) * 4)]


@pytest.mark.parametrize("system,nx,ny,bc", CASES2)
def test_marching_strips(system, nx, ny, bc):
    require_gpu()
    p = _tall(system, nx, ny, bc, 12)
    assert _rows_of(p, A.F32) == 0 and _rows_of(p, A.F64) == 0
    say(f"[marching strips {system} {nx}x{ny} bc={bc}]")
    first, Lo = oracle_run(p, 1, parallel=True), oracle_run(p, p.steps, parallel=True)
    G = gpu_lattice(p, A.F64, omega_export=True)
    G.step(p.steps)
    st = G.sync(check=False)
    assert fp64_parity_ok(G.moments(), Lo.moments(), p.system)
    if p.system != A.REACTIVE:
        assert st["t"] == Lo.t and np.array_equal(G.omega(), Lo.last_omega())
    G.close()
    G = gpu_lattice(p, A.F32, omega_export=True)
    G.step(1)
    assert np.max(np.abs(G.omega() - first.last_omega())) <= TOL_OMEGA32_1
    G.step(p.steps - 1)
    U = G.moments()
    G.close()
    assert rel_l1(U, Lo.moments()) <= TOL_FP32
    assert np.array_equal(U, _served(p, p.steps))


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system,nx", [("euler", 250), ("swe", 250), ("swe", 249), ("advection", 250), ("reactive", 118)])
def test_march_takes_null_steps(system, nx, prec):
    """A time-targeted run, whose surplus launches copy the state, equals
    stepping exactly."""
    require_gpu()
    p = _tall(system, nx, {"swe": 2060, "reactive": 1900}.get(system, 1090), (T,) * 4, 0)
    assert _rows_of(p, prec) == 0
    a, b = (gpu_lattice(p, prec) for _ in range(2))
    a.step(5)
    st = a.sync(check=False)
    k = a.step_until(st["t"] + 6.5 * st["last_dt"])
    b.step(5 + k)
    say(f"[march, null steps] {system} {nx}x{p.ny} prec={prec}: {k} steps")
    assert a.sync(check=False) == b.sync(check=False) and np.array_equal(a.moments(), b.moments())
    a.step(2)
    b.step(2)
    assert np.array_equal(a.moments(), b.moments())
    a.close()
    b.close()


def _pads_untouched(p, prec, q):
    """Steps on population buffers filled with a byte pattern change no byte
    outside the cells of their planes."""
    cfg = A.config_from(p, precision=prec)
    L = A.Lattice(cfg, owner="torch")
    size, cells = (8 if prec == A.F64 else 4), p.cells
    # the binding allocates f[0], u[0], f[1], u[1], each at a 256-byte aligned
    # offset of its tensor
    views = [t[(-t.data_ptr()) % 256:][:L.sizes.f_bytes] for t in (L._tensors[0], L._tensors[2])]
    views[0].fill_(SENTINEL)
    L.set_state(p.U0, p.bed)
    views[1].fill_(SENTINEL)  # f[1] holds nothing before the first step
    L.step(7)
    L.sync(check=False)
    ps, n = (cells + 63) // 64 * 64 + 1088, q * L.m
    ok = True
    for v in views:
        raw = v.cpu().numpy()
        ok = ok and bool(np.all(raw[:n * ps * size].reshape(n, ps * size)[:, cells * size:] == SENTINEL))
        ok = ok and bool(np.all(raw[n * ps * size:] == SENTINEL))
    U = L.moments()
    L.close()
    ref = gpu_lattice(p, prec)
    ref.step(7)
    same = np.array_equal(U, ref.moments())
    ref.close()
    return ok and same


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system,nx,ny,bc", [CASES2[i] for i in (1, 3, 6, 8, 11, 13, 14)])
def test_marching_strips_write_only_lattice_cells(system, nx, ny, bc, prec):
    require_gpu()
    say(f"[march, pads] {system} {nx}x{ny} prec={prec}")
    assert _pads_untouched(_tall(system, nx, ny, bc, 0), prec, 5)


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system,nx,h,k,xbc", [("advection", 250, 128, 10, T), ("euler", 250, 100, 12, T),
                                               ("euler", 59, 60, 46, R), ("swe", 250, 128, 18, R),
                                               ("swe", 249, 90, 24, T), ("reactive", 118, 90, 21, R),
                                               ("euler", 200, 101, 14, P)])
def test_march_gives_the_bits_of_tiles_2d(system, nx, h, k, xbc, prec):
    """h rows, periodic in y, in tiles; the same k times over, marching."""
    require_gpu()
    p = crop(MAKE2[system](), nx, h, bc=(xbc, xbc, P, P), ox=(256 - nx) // 2, oy=60)
    q = dataclasses.replace(p, ny=k * h, y1=p.y0 + k * (p.y1 - p.y0), U0=np.tile(p.U0, (1, k, 1)),
                            bed=None if p.bed is None else np.tile(p.bed, (k, 1)))
    assert _rows_of(p, prec) > 0 and _rows_of(q, prec) == 0
    a, b = (gpu_lattice(x, prec, omega_export=True) for x in (p, q))
    a.step(20)
    b.step(20)
    say(f"[march == tiles] {system} {nx}x{h} x{k} prec={prec}")
    sa, sb = a.sync(check=False), b.sync(check=False)
    assert sa == sb
    assert np.array_equal(np.tile(a.moments(), (1, k, 1)), b.moments())
    assert np.array_equal(np.tile(a.omega(), (k, 1)), b.omega())
    a.close()
    b.close()


def test_reactive_tiles_beside_a_large_lattice():
    """FP32 512^2 reactive Euler: 468 tiles alone, strips beside a lattice too
    large for tiles."""
    require_gpu()
    p = W.reactive_seeded_2d(0, n=512, steps=20)
    assert _rows_of(p) > 0
    G = gpu_lattice(p, A.F32)
    G.step(p.steps)
    say("[tiles reactive 512^2]")
    assert np.array_equal(G.moments(), _served_beside(p, LARGE))
    G.close()


# more than one tile per CU, and the last and first heights on both sides of the
# tiles' line (8 strips of Euler: 672 rows; 13 of shallow water: 780)
@pytest.mark.parametrize("system,nx,ny,bc,tiled", [
    ("euler", 400, 397, (T,) * 4, True), ("euler", 601, 433, (R,) * 4, True), ("euler", 601, 433, (P, P, T, R), True),
    ("advection", 512, 512, (P,) * 4, True), ("advection", 400, 397, (T, T, P, P), True),
    ("reactive", 400, 397, (T, R, R, T), True), ("swe", 700, 700, (R,) * 4, True), ("swe", 601, 433, (P, P, T, R), True),
    ("euler", 464, 672, (T, R, P, P), True), ("euler", 464, 673, (T, R, P, P), False),
    ("swe", 754, 780, (R,) * 4, True), ("swe", 754, 781, (R,) * 4, False)])
def test_many_tiles_against_oracle_and_served(system, nx, ny, bc, tiled):
    require_gpu()
    n = max(nx, ny)
    make = {"advection": lambda: W.advection_sine_2d(n=n, ax=0.8, ay=-0.5), "euler": lambda: W.euler_seeded_2d(4, n=n),
            "swe": lambda: W.swe_bed_2d(1, n=n), "reactive": lambda: W.reactive_seeded_2d(1, n=n)}[system]
    p = crop(make(), nx, ny, bc=bc, ox=(n - nx) // 2, oy=(n - ny) // 2, steps=6)
    rows = _rows_of(p)
    assert (rows > 0) == tiled and rows == _rows_of(p, A.F64)
    if tiled:
        assert -(-nx // 58) * -(-ny // (rows - 6)) > 256
    say(f"[many tiles {system} {nx}x{ny} bc={bc}] tiles of {rows} rows")
    Lo = oracle_run(p, p.steps, parallel=True)
    G = gpu_lattice(p, A.F64, omega_export=True)
    G.step(p.steps)
    st = G.sync(check=False)
    assert fp64_parity_ok(G.moments(), Lo.moments(), p.system)
    if p.system != A.REACTIVE:
        assert st["t"] == Lo.t and np.array_equal(G.omega(), Lo.last_omega())
    G.close()
    G = gpu_lattice(p, A.F32)
    G.step(p.steps)
    U = G.moments()
    assert rel_l1(U, Lo.moments()) <= TOL_FP32
    assert np.array_equal(U, _served_beside(p, LARGE))
    G.close()


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system,nx,ny,bc", [("euler", 400, 397, (T,) * 4), ("swe", 601, 433, (P, P, T, R)),
                                             ("reactive", 400, 397, (T, R, R, T)), ("advection", 401, 512, (T,) * 4)])
def test_many_tiles_write_only_lattice_cells(system, nx, ny, bc, prec):
    require_gpu()
    p = crop({"advection": W.advection_sine_2d, "euler": W.euler_seeded_2d, "swe": W.swe_bed_2d,
              "reactive": W.reactive_seeded_2d}[system](n=640), nx, ny, bc=bc, ox=20, oy=20)
    assert _rows_of(p, prec) > 0
    say(f"[many tiles, pads] {system} {nx}x{ny} prec={prec}")
    assert _pads_untouched(p, prec, 5)


def _box(system, nx, ny, nz, bc, steps):
    """An nx x ny x nz box: the cube's middle columns, its planes walked there
    and back."""
    n = 72
    p = MAKE3[system](n=n)
    dx, ox, oy = (p.x1 - p.x0) / n, (n - nx) // 2, (n - ny) // 2
    U0 = p.U0[:, :, oy:oy + ny, ox:ox + nx][:, _there_and_back(nz, n)]
    return dataclasses.replace(p, nx=nx, ny=ny, nz=nz, x0=0.0, x1=nx * dx, y0=0.0, y1=ny * dx, z0=0.0, z1=nz * dx,
                               U0=np.ascontiguousarray(U0), bc=tuple(bc[:4]), bc_z=tuple(bc[4:]), steps=steps)


# past the tiles' line (5 per CU, advection 16): ragged in every axis, planes in
# many chunks; and two lattices on either side of it
CASES3 = [("euler", 13, 11, 2605, (T,) * 6), ("euler", 33, 17, 700, (R, T, P, P, T, R)), ("euler", 70, 37, 233, (P, P, R, R, P, P)),
          ("advection", 13, 11, 8203, (P,) * 6), ("advection", 33, 17, 2191, (T, T, P, P, T, T)),
          ("reactive", 13, 11, 2605, (R, R, T, R, P, P)), ("reactive", 33, 17, 700, (T,) * 6), ("reactive", 70, 37, 233, (R,) * 6)]


@pytest.mark.parametrize("system,nx,ny,nz,bc", CASES3)
def test_marching_planes(system, nx, ny, nz, bc):
    """Steps, the omega export, surplus launches of a time-targeted run, and
    steps after them."""
    require_gpu()
    p = _box(system, nx, ny, nz, bc, 4)
    assert _rows_of(p, A.F32) == 0 and _rows_of(p, A.F64) == 0
    say(f"[marching planes {system} {nx}x{ny}x{nz} bc={bc}]")
    Lo = oracle_run(p, p.steps, parallel=True)
    G = gpu_lattice(p, A.F64, omega_export=True)
    G.step(p.steps)
    st = G.sync(check=False)
    assert fp64_parity_ok(G.moments(), Lo.moments(), p.system)
    if p.system != A.REACTIVE:
        assert st["t"] == Lo.t and np.array_equal(G.omega(), Lo.last_omega())
    k = G.step_until(st["t"] + 2.5 * st["last_dt"])
    G.step(1)
    Lo.run(k + 1)
    assert fp64_parity_ok(G.moments(), Lo.moments(), p.system)
    G.close()
    G = gpu_lattice(p, A.F32)
    G.step(p.steps + k + 1)
    assert rel_l1(G.moments(), Lo.moments()) <= TOL3[system]
    G.close()


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system,nx,ny,nz,bc", [CASES3[i] for i in (1, 4, 7)])
def test_marching_planes_write_only_lattice_cells(system, nx, ny, nz, bc, prec):
    require_gpu()
    say(f"[marching planes, pads] {system} {nx}x{ny}x{nz} prec={prec}")
    assert _pads_untouched(_box(system, nx, ny, nz, bc, 0), prec, 7)


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system,nx,ny,h,k,bc", [("euler", 33, 17, 24, 30, (T, R, P, P)), ("euler", 70, 37, 16, 15, (R,) * 4),
                                                 ("advection", 33, 17, 40, 55, (T, T, P, P)),
                                                 ("reactive", 33, 17, 24, 30, (T, R, R, T)),
                                                 ("reactive", 70, 37, 16, 15, (P,) * 4),
                                                 ("euler", 70, 37, 64, 4, (T, R, P, P)),
                                                 ("reactive", 70, 37, 64, 4, (R, T, R, T))])
def test_march_gives_the_bits_of_tiles_3d(system, nx, ny, h, k, bc, prec):
    """h planes, periodic in z, in tiles (low ones, and full ones of 64 planes);
    the same k times over, marching."""
    require_gpu()
    p = _box(system, nx, ny, 72, bc + (P, P), 0)
    o, dz = (72 - h) // 2, p.z1 / 72
    p = dataclasses.replace(p, nz=h, z1=h * dz, U0=np.ascontiguousarray(p.U0[:, o:o + h]))
    q = dataclasses.replace(p, nz=k * h, z1=k * h * dz, U0=np.tile(p.U0, (1, k, 1, 1)))
    assert _rows_of(p, prec) > 0 and _rows_of(q, prec) == 0
    a, b = (gpu_lattice(x, prec, omega_export=True) for x in (p, q))
    a.step(8)
    b.step(8)
    say(f"[march == tiles] {system} {nx}x{ny}x{h} x{k} prec={prec}")
    assert a.sync(check=False) == b.sync(check=False)
    assert np.array_equal(np.tile(a.moments(), (1, k, 1, 1)), b.moments())
    assert np.array_equal(np.tile(a.omega(), (k, 1, 1)), b.omega())
    a.close()
    b.close()


@pytest.mark.parametrize("system,nz", [("euler", 96), ("euler", 104), ("reactive", 104)])
def test_both_sides_of_five_tiles_per_cu(system, nz):
    """80 x 80 columns: 1200 tiles, and 1300 where the march takes over."""
    require_gpu()
    n = 104
    p = MAKE3[system](n=n)
    dx, o = (p.x1 - p.x0) / n, (n - 80) // 2
    p = dataclasses.replace(p, nx=80, ny=80, nz=nz, x0=0.0, x1=80 * dx, y0=0.0, y1=80 * dx, z0=0.0, z1=nz * dx, steps=4,
                            U0=np.ascontiguousarray(p.U0[:, :nz, o:o + 80, o:o + 80]))
    assert (_rows_of(p) > 0) == (nz == 96)
    say(f"[five tiles per CU] {system} 80x80x{nz}")
    Lo = oracle_run(p, 4, parallel=True)
    G = gpu_lattice(p, A.F64)
    G.step(4)
    assert fp64_parity_ok(G.moments(), Lo.moments(), p.system)
    G.close()
    G = gpu_lattice(p, A.F32)
    G.step(4)
    assert rel_l1(G.moments(), Lo.moments()) <= TOL3[system]
    G.close()


def test_fp64_advection_beyond_4_gib():
    """FP64 advection, two columns per lane, with population buffers beyond 4
    GiB (64-bit addresses in place of buffer resources): a periodic lattice
    and the same 26 x 26 times over take the same steps."""
    require_gpu()
    p = crop(W.advection_sine_2d(n=400, ax=0.8, ay=-0.5), 400, 400, bc=(P,) * 4)
    k = 26
    q = dataclasses.replace(p, nx=k * p.nx, ny=k * p.ny, x1=p.x0 + k * (p.x1 - p.x0), y1=p.y0 + k * (p.y1 - p.y0),
                            U0=np.tile(p.U0, (1, k, k)))
    assert A.query_sizes(A.config_from(q, precision=A.F64)).f_bytes > 1 << 32
    say(f"[march, beyond 4 GiB] advection {q.nx}^2 FP64")
    a, b = (gpu_lattice(x, A.F64) for x in (p, q))
    a.step(3)
    b.step(3)
    assert a.sync() == b.sync()
    U = b.moments()
    b.close()
    assert np.array_equal(np.tile(a.moments(), (1, k, k)), U)
    a.close()
