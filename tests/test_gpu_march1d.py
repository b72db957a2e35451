"""The one-workgroup march of small 1D lattices (state in registers, halos and
bounds through LDS) against one launch per step, bit for bit: sizes where the
deal of cells to waves and lanes can go wrong (one wave, the first cell of a
second wave, the last size of one and of two cells per lane, too large for the
march), every face, and time-targeted runs that stop inside a launch."""
import numpy as np
import pytest

from paper_2609_18177_amd import arlbm as A
from paper_2609_18177_amd import workloads as W
from gpu_common import gpu_lattice, require_gpu, say

pytestmark = pytest.mark.gpu

SIZES = (4, 5, 7, 58, 59, 117, 927, 928, 929, 1045, 1920, 1921)


def _problem(kind, n, face):
    p = {"advection": lambda: W.advection_sine(n=n), "euler": lambda: W.euler_seeded_1d(3, n=n),
         "swe": lambda: W.swe_bed_1d(n=n), "reactive": lambda: W.reactive_seeded_1d(1, n=n)}[kind]()
    p.bc = (face,) * 4
    return p


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("kind,face", [("advection", A.PERIODIC), ("advection", A.TRANSMISSIVE),
                                       ("euler", A.REFLECTIVE), ("euler", A.PERIODIC), ("swe", A.REFLECTIVE),
                                       ("swe", A.TRANSMISSIVE), ("reactive", A.TRANSMISSIVE),
                                       ("reactive", A.REFLECTIVE)])
def test_march_equals_single_steps(kind, face, prec):
    require_gpu()
    for n in SIZES:
        p = _problem(kind, n, face)
        say(f"[march {kind} face={face} prec={prec}] {n} cells")
        a, b = (gpu_lattice(p, prec, omega_export=True) for _ in range(2))
        a.step(21)
        for _ in range(21):
            b.step(1)
        sa, sb = a.sync(check=False), b.sync(check=False)
        assert np.array_equal(a.moments(), b.moments()) and np.array_equal(a.omega(), b.omega()), n
        assert sa == sb, n
        # to a time inside the next launch of the march: surplus steps change nothing
        goal = sa["t"] + 4.5 * sa["last_dt"]
        taken = a.step_until(goal)
        k = 0
        while b.sync(check=False)["t"] < goal:
            b.step(1)
            k += 1
        sa, sb = a.sync(check=False), b.sync(check=False)
        assert taken == k and sa == sb, n
        assert np.array_equal(a.moments(), b.moments()), n
        a.step(3)
        b.step(1)
        b.step(1)
        b.step(1)
        assert np.array_equal(a.moments(), b.moments()), n
        a.close()
        b.close()
