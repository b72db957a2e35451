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


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("system", ["euler", "swe", "reactive"])
def test_tiles_without_a_step(system, prec):
    """Launches that take no step: at the stop time the state carries over;
    with wave-speed bounds of zero (every density NaN) the degenerate flag is
    raised, at the stop time too."""
    require_gpu()
    p = crop(MAKE[system](), 70, 41, bc=(T,) * 4, ox=93, oy=107, steps=1)
    G = gpu_lattice(p, prec)
    G.step(3)
    st = G.sync(check=False)
    assert G.step_until(st["t"] + 0.5 * st["last_dt"]) == 1  # and one launch at the stop time
    H = gpu_lattice(p, prec)
    H.step(4)
    assert G.sync(check=False) == H.sync(check=False) and np.array_equal(G.moments(), H.moments())
    H.close()
    st = G.sync(check=False)
    blob = bytearray(G.save_state())
    real = np.float32 if prec == A.F32 else np.float64
    cells = np.full(p.nx * p.ny, np.nan, dtype=real).tobytes()
    blob[56:56 + len(cells)] = cells  # f_0 of the first field, after the header
    G.load_state(bytes(blob))
    say(f"[no step {system} prec={prec}]")
    # a step to NaN, and a launch that is flagged, so not counted as at the stop time
    assert G.step_until(st["t"] + 0.5 * st["last_dt"], max_steps=2) == 2
    bad = G.sync(check=False)
    assert bad["flags"] & A.FLAG_NONFINITE and bad["flags"] & A.FLAG_DEGENERATE
    assert bad["first_bad_step"] == 4 and bad["step"] == 6
    G.close()
