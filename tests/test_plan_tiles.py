"""Which lattices are stepped in tiles (host logic, no GPU): the 2D rule on
both sides of its line and over sizes, the 3D rule, and the server's choice."""
import random

import numpy as np
import pytest

from paper_2609_18177_amd import arlbm as A

CUS = 256


def _cfg(system, n, precision=A.F32):
    """A lattice of n = (nx[, ny[, nz]]) cells of spacing 1."""
    n = tuple(n)
    nx, ny, nz = n + (1,) * (3 - len(n))
    return A.config_from(None, precision=precision, system=system, dim=len(n), nx=nx, ny=ny, nz=nz, x0=0.0, x1=float(nx),
                         y0=0.0, y1=float(ny), z0=0.0, z1=float(nz))


def _rows(system, nx, ny):
    """The rule: the rows of a tile (8 to 16, 6 of them halo) with the fewest
    waves per CU, at most 40, 64 for shallow water; the lowest of equals."""
    line = 64 if system == A.SWE else 40
    best = [0, line]
    for rows in range(16, 7, -1):
        tiles = -(-nx // 58) * -(-ny // (rows - 6))
        waves = rows * -(-tiles // CUS)
        if waves <= best[1]:
            best = [rows, waves]
    return best


@pytest.mark.parametrize("precision", [A.F32, A.F64])
@pytest.mark.parametrize("system", [A.ADVECTION, A.EULER, A.SWE, A.REACTIVE])
def test_rule_in_2d(system, precision):
    rng = random.Random(11)
    sizes = [(4, 4), (58, 8), (256, 256), (512, 512), (601, 433), (700, 700), (2048, 2048), (58, 5376), (58, 5377)]
    sizes += [(rng.randint(4, 1200), rng.randint(4, 1200)) for _ in range(200)]
    got = A.plan_tiles([_cfg(system, n, precision) for n in sizes], CUS)[0]
    assert [int(g) for g in got] == [_rows(system, *n)[0] for n in sizes]


def test_line_in_2d():
    """One strip: 13 rows at three tiles per CU are the last 39 waves; shallow
    water: 16 rows at four the last 64."""
    for system, last in ((A.EULER, 5376), (A.SWE, 10240)):
        alone, _ = A.plan_tiles([_cfg(system, (58, last)), _cfg(system, (58, last + 1))], CUS)
        assert alone[0] > 0 and alone[1] == 0


@pytest.mark.parametrize("system,precision,per_cu,tz", [(A.EULER, A.F32, 5, 8), (A.EULER, A.F64, 5, 8),
                                                        (A.ADVECTION, A.F32, 16, 8), (A.ADVECTION, A.F64, 16, 8),
                                                        (A.REACTIVE, A.F32, 5, 8), (A.REACTIVE, A.F64, 5, 4)])
def test_rule_in_3d(system, precision, per_cu, tz):
    """Low tiles up to one per CU, then tiles up to per_cu per CU."""
    n = [(8, 8, 4 * CUS), (8, 8, 4 * CUS + 1), (8, 8, tz * per_cu * CUS), (8, 8, tz * per_cu * CUS + 1), (24, 24, 24),
         (256, 256, 256)]
    alone, served = A.plan_tiles([_cfg(system, k, precision) for k in n], CUS)
    assert list(alone) == [4, tz, tz, 0, 4, 0] and list(served) == list(alone)


def test_few_and_small_2d_lattices_of_a_server():
    e, s = (lambda *n: _cfg(A.EULER, n)), (lambda *n: _cfg(A.SWE, n))
    one_d = _cfg(A.EULER, (20000,))
    cube = _cfg(A.EULER, (40, 40, 40))

    def served(*cfgs):
        return [int(v) for v in A.plan_tiles(list(cfgs), CUS)[1]]

    r = _rows(A.EULER, 256, 256)
    assert r[1] == 12
    assert served(e(256, 256)) == [r[0]]                                   # 12 + 8 of 48
    assert served(e(256, 256), e(256, 256)) == [r[0]] * 2                  # 40 of 48
    assert served(e(256, 256), e(256, 256), e(256, 256)) == [0] * 3        # 60
    assert served(e(256, 256), one_d) == [r[0], 0]                         # 20 + 12
    assert served(e(256, 256), e(256, 256), one_d) == [0, 0, 0]            # 40 + 12
    assert served(cube, e(256, 256)) == [8 if A.plan_tiles([cube], CUS)[0][0] == 8 else 4, r[0]]
    assert served(e(256, 256), e(1000, 1000)) == [0, 0]                    # one of them marches
    assert served(s(600, 600)) == [_rows(A.SWE, 600, 600)[0]]
    assert served(s(600, 600), e(64, 64)) == [0, 0]                        # Euler's lower line
    assert served(one_d) == [0] and served() == []


def test_bad_arguments():
    for cfgs, cus in (([_cfg(A.EULER, (64, 64))], 0), ([_cfg(A.EULER, (64, 3))], CUS)):
        with pytest.raises(A.ArlbmError) as err:
            A.plan_tiles(cfgs, cus)
        assert err.value.code == A.EINVAL
