"""The tiled 2D step of small lattices (one wave per row of a tile) against the
oracle and against the batched server's marching strips: FP64 bit for bit (the
reactive system within the pointwise bound of its two independent root
finders), FP32 the same bits as served beside a large lattice (the batched
launch steps both) and as served alone (the server steps it in tiles).  Sizes at the edges of the
tiles: fewer cells than a halo is wide, one column or row more than a tile's,
several tiles with ragged ends."""
import numpy as np
import pytest

from paper_2609_18177_amd import arlbm as A
from paper_2609_18177_amd import workloads as W
from gpu_common import fp64_parity_ok, gpu_lattice, oracle_run, require_gpu, say
from test_gpu_strips import _served, crop

pytestmark = pytest.mark.gpu

T, R, P = A.TRANSMISSIVE, A.REFLECTIVE, A.PERIODIC
MAKE = {"advection": lambda: W.advection_sine_2d(n=256, ax=0.8, ay=-0.5), "euler": lambda: W.euler_seeded_2d(4, n=256),
        "swe": lambda: W.swe_bed_2d(1, n=256), "reactive": lambda: W.reactive_seeded_2d(1, n=256)}


def _served_beside(p, large):
    """p's result from a server that steps it beside a lattice too large for tiles."""
    srv = A.Server(1 << 30, A.F32)
    srv.submit(A.config_from(large, precision=A.F32), large.U0, large.bed, p.steps + 1)
    rid = srv.submit(A.config_from(p, precision=A.F32), p.U0, p.bed, p.steps)
    done = {}
    while rid not in done:
        srv.iterate(4)
        done.update({c["id"]: c for c in srv.poll(4)})
    srv.close()
    assert done[rid]["status"] == 0
    return done[rid]["U"].reshape((-1, p.ny, p.nx))


LARGE = W.euler_seeded_2d(0, n=800)


@pytest.mark.parametrize("nx,ny", [(4, 4), (58, 6), (59, 7), (116, 10), (117, 33), (200, 101), (250, 256)])
@pytest.mark.parametrize("system,bc", [("advection", (P,) * 4), ("advection", (T, T, P, P)), ("euler", (T,) * 4),
                                       ("euler", (R, T, P, P)), ("swe", (R,) * 4), ("swe", (P, P, T, R)),
                                       ("reactive", (T, R, R, T))])
def test_tiles_against_oracle_and_served(system, bc, nx, ny):
    require_gpu()
    p = crop(MAKE[system](), nx, ny, bc=bc, ox=(256 - nx) // 2, oy=(256 - ny) // 2, steps=12)
    say(f"[tiles {system} {nx}x{ny} bc={bc}]")
    Lo = oracle_run(p, p.steps)
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
    assert np.array_equal(U, _served_beside(p, LARGE)) and np.array_equal(U, _served(p, p.steps))
    G.close()
