"""The tiled 3D step of small lattices against the oracle: FP64 bit for bit (the
reactive system within the pointwise bound of its two independent root
finders), FP32 within the 3D bound.  Both tile heights (the low tiles hold
lattices of up to one tile per CU), fewer cells than a halo is wide, one cell
more than a tile, every face, and a time-targeted run that ends in surplus
launches."""
import numpy as np
import pytest

from paper_2609_18177_amd import arlbm as A
from paper_2609_18177_amd import workloads as W
from gpu_common import fp64_parity_ok, gpu_lattice, oracle_run, rel_l1, require_gpu, say
from test_gpu_3d import TOL_FP32

pytestmark = pytest.mark.gpu

T, R, P = A.TRANSMISSIVE, A.REFLECTIVE, A.PERIODIC


def _window(p, nx, ny, nz, bc):
    """The nx x ny x nz corner of a cube around its centre, with other faces."""
    dx = (p.x1 - p.x0) / p.nx
    o = [(p.nx - n) // 2 for n in (nx, ny, nz)]
    p.U0 = np.ascontiguousarray(p.U0[:, o[2]:o[2] + nz, o[1]:o[1] + ny, o[0]:o[0] + nx])
    p.nx, p.ny, p.nz = nx, ny, nz
    p.x0, p.x1, p.y0, p.y1, p.z0, p.z1 = 0.0, nx * dx, 0.0, ny * dx, 0.0, nz * dx
    p.bc, p.bc_z = tuple(bc[:4]), tuple(bc[4:])
    return p


# (4 x 8 x 9 .. 33 x 40 x 17: low tiles; 60 x 57 x 41: full ones, 8 x 8 x 6 of them)
@pytest.mark.parametrize("n", [(4, 8, 9), (8, 4, 4), (9, 17, 5), (33, 40, 17), (60, 57, 41)])
@pytest.mark.parametrize("system,bc", [("advection", (P,) * 6), ("advection", (T, T, P, P, T, T)), ("euler", (T,) * 6),
                                       ("euler", (R, T, P, P, T, R)), ("euler", (P, P, R, R, P, P)),
                                       ("reactive", (R, R, T, R, P, P)), ("reactive", (T,) * 6)])
def test_tiles_against_oracle(system, bc, n):
    require_gpu()
    p = _window({"advection": W.advection_sine_3d, "euler": W.euler_octants_3d, "reactive": W.reactive_sphere_3d}[system](n=60),
                *n, bc)
    say(f"[3d tiles {system} {n} bc={bc}]")
    Lo = oracle_run(p, 6, parallel=True)
    G = gpu_lattice(p, A.F64, omega_export=True)
    G.step(6)
    st = G.sync(check=False)
    assert fp64_parity_ok(G.moments(), Lo.moments(), p.system)
    if p.system != A.REACTIVE:
        assert st["t"] == Lo.t and np.array_equal(G.omega(), Lo.last_omega())
    k = G.step_until(st["t"] + 2.5 * st["last_dt"])
    Lo.run(k)
    assert fp64_parity_ok(G.moments(), Lo.moments(), p.system)
    G.close()
    G = gpu_lattice(p, A.F32)
    G.step(6 + k)
    assert rel_l1(G.moments(), Lo.moments()) < TOL_FP32
    G.close()
