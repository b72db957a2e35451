"""The march of 1D lattices in registers (halos and bounds through LDS in one
workgroup, through memory between several) against one launch per step, bit for
bit: sizes where the deal of cells to waves, lanes and workgroups can go wrong
(one wave, the first cell of a second wave, the last size of one and of two
cells per lane, two workgroups, one more than a workgroup's waves, more bounds
than lanes, five waves a workgroup), every face, time-targeted runs that stop
inside a launch, several lattices on streams of their own, and a captured
stream, where the steps are launched one by one."""
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


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("kind,face", [("advection", A.PERIODIC), ("euler", A.REFLECTIVE), ("euler", A.PERIODIC),
                                       ("swe", A.REFLECTIVE), ("reactive", A.TRANSMISSIVE)])
def test_march_over_several_workgroups(kind, face, prec):
    require_gpu()
    # 15000 cells: 65 workgroups, more than lanes; 60000 in FP32: 1035 waves, five a workgroup
    for n in (407, 697, 929, 1921, 4096, 15000, 60000):
        p = _problem(kind, n, face)
        say(f"[grid march {kind} face={face} prec={prec}] {n} cells")
        a, b = (gpu_lattice(p, prec) for _ in range(2))
        a.step(35)
        for _ in range(35):
            b.step(1)
        sa, sb = a.sync(check=False), b.sync(check=False)
        assert sa == sb and np.array_equal(a.moments(), b.moments()), n
        goal = sa["t"] + 40.5 * sa["last_dt"]
        k = a.step_until(goal)
        a.step(33)
        for _ in range(k + 33):
            b.step(1)
        sa, sb = a.sync(check=False), b.sync(check=False)
        assert sa == sb and np.array_equal(a.moments(), b.moments()), n
        a.close()
        b.close()


def test_march_on_several_streams():
    """Lattices stepped at the same time on streams of their own."""
    import torch

    require_gpu()
    ps = [_problem("euler", n, A.TRANSMISSIVE) for n in (4096, 9000, 30000, 2000, 14000, 50000)]
    want, got, lats = [], [], []
    for p in ps:
        L = gpu_lattice(p, A.F32)
        for _ in range(200):
            L.step(1)
        want.append(L.moments())
        L.close()
    for p in ps:
        L = A.Lattice(A.config_from(p, precision=A.F32), stream=torch.cuda.Stream())
        L.set_state(p.U0)
        lats.append(L)
    for _ in range(4):
        for L in lats:
            L.step(50)
    got = [L.moments() for L in lats]
    say("[grid march] six streams", [bool(np.array_equal(a, b)) for a, b in zip(got, want)])
    assert all(np.array_equal(a, b) for a, b in zip(got, want))


def test_march_in_a_captured_stream():
    """Steps recorded into a graph run when it is launched, as one launch per step."""
    import torch

    require_gpu()
    p = _problem("euler", 4096, A.TRANSMISSIVE)
    ref = gpu_lattice(p, A.F32)
    ref.step(40)
    want = ref.moments()
    ref.close()
    s = torch.cuda.Stream()
    L = A.Lattice(A.config_from(p, precision=A.F32), stream=s)
    L.set_state(p.U0)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        L.step(40)
    g.replay()
    torch.cuda.synchronize()
    assert np.array_equal(L.moments(), want)
    L.close()


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("kind", ["euler", "swe", "reactive"])
def test_time_target_from_the_initial_state(kind, prec):
    """From a state no step was taken from, the length of the first launch
    comes from the initial wave speeds, with half as many steps in reserve:
    the last launch ends at the target, inside it, and a cap on the steps
    falls before or inside the reserve.  928 cells: the march's last size."""
    require_gpu()
    for n in (4, 59, 928):
        p = _problem(kind, n, A.REFLECTIVE)
        say(f"[march to a time {kind} prec={prec}] {n} cells")
        a, b, c = (gpu_lattice(p, prec) for _ in range(3))
        b.step(1)
        goal = 60.5 * b.sync(check=False)["last_dt"]
        k = 1
        while k < 500 and b.sync(check=False)["t"] < goal:
            b.step(1)
            k += 1
        assert a.step_until(goal) == k, n
        sa, sb = a.sync(check=False), b.sync(check=False)
        assert sa == sb and np.array_equal(a.moments(), b.moments()), n
        assert c.step_until(goal, max_steps=k - 1) == k - 1, n
        assert c.step_until(goal, max_steps=k + 9) == 1, n
        assert c.sync(check=False) == sb and np.array_equal(c.moments(), b.moments()), n
        for x in (a, b, c):
            x.close()
