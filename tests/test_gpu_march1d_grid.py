"""The march of 1D lattices over several workgroups where its launches do not
take all the steps they were made for, bit for bit against one launch per
step."""
import numpy as np
import pytest

from paper_2609_18177_amd import arlbm as A
from paper_2609_18177_amd import workloads as W
from gpu_common import gpu_lattice, require_gpu, say

pytestmark = pytest.mark.gpu


def _hump(n):
    """A pressure hump of ten cells, whose two halves run apart: the time step
    grows by a third within a few steps, so a run of t needs about three
    quarters of the steps that its first time step promises."""
    p = W.euler_riemann_1d(*W.SOD, n=n, cfl=0.5)
    x = (np.arange(n) + 0.5 - n / 2) / 10.0
    p.U0 = np.stack([np.ones(n), np.zeros(n), (1.0 + 9.0 * np.exp(-x * x)) / 0.4])
    return p


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("n", [929, 4096, 15000])
def test_launches_that_take_no_step(n, prec):
    """A run to a time that is enqueued as 1024 + r steps and needs fewer than
    1024: its second launch takes none, for r of every remainder modulo the
    three slots that bounds and times take in turn."""
    require_gpu()
    for r in (1, 2, 3, 4, 35):
        p = _hump(n)
        say(f"[grid march, no step] {n} cells prec={prec} r={r}")
        a, b = (gpu_lattice(p, prec) for _ in range(2))
        dt0 = p.cfl * (p.x1 - p.x0) / n / a.sync()["abar"][0]
        goal = (1022.5 + r) * dt0
        taken = a.step_until(goal)
        k = 0
        while k < 1024 and b.sync(check=False)["t"] < goal:
            b.step(1)
            k += 1
        sa, sb = a.sync(), b.sync()
        assert 0 < taken == k < 1024
        assert sa == sb and sa["flags"] == 0 and np.array_equal(a.moments(), b.moments())
        assert a.step_until(goal) == 0
        a.step(35)
        for _ in range(35):
            b.step(1)
        assert a.sync() == b.sync() and np.array_equal(a.moments(), b.moments())
        a.close()
        b.close()


def _problem(kind, n, face):
    p = {"advection": lambda: W.advection_sine(n=n), "euler": lambda: W.euler_seeded_1d(3, n=n),
         "swe": lambda: W.swe_bed_1d(n=n), "reactive": lambda: W.reactive_seeded_1d(1, n=n)}[kind]()
    p.bc = (face,) * 4
    return p


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("kind,face", [("advection", A.PERIODIC), ("euler", A.REFLECTIVE), ("swe", A.REFLECTIVE),
                                       ("swe", A.TRANSMISSIVE), ("reactive", A.TRANSMISSIVE)])
def test_launch_whose_workgroups_do_not_all_run(kind, face, prec):
    """With no look at the others a launch calls its march off, and one
    workgroup takes its steps: fewer strips than its waves, as many and more,
    whole launches, time-targeted ones, and the march again after them."""
    require_gpu()
    for n in (697, 929, 1921, 4096):
        p = _problem(kind, n, face)
        say(f"[grid march, called off] {kind} face={face} prec={prec} {n} cells")
        a, b = (gpu_lattice(p, prec, omega_export=True) for _ in range(2))
        a.set_march_limits(gather_looks=0)
        a.step(35)
        for _ in range(35):
            b.step(1)
        sa, sb = a.sync(check=False), b.sync(check=False)
        assert sa == sb and np.array_equal(a.moments(), b.moments()) and np.array_equal(a.omega(), b.omega()), n
        k = a.step_until(sa["t"] + 40.5 * sa["last_dt"])
        a.set_march_limits()
        a.step(33)
        for _ in range(k + 33):
            b.step(1)
        assert a.sync(check=False) == b.sync(check=False) and np.array_equal(a.moments(), b.moments()), n
        a.close()
        b.close()


def test_march_limits_are_checked():
    require_gpu()
    L = gpu_lattice(_problem("euler", 4096, A.TRANSMISSIVE), A.F32)
    for bad in ((-1, 1), (1, -1)):
        with pytest.raises(A.ArlbmError) as e:
            L.set_march_limits(*bad)
        assert e.value.code == A.EINVAL
    L.close()


@pytest.mark.parametrize("n,prec", [(4096, A.F32), (4096, A.F64), (15000, A.F32)])
def test_lattices_on_several_streams_run_side_by_side(n, prec):
    """Four lattices on streams of their own take less than three times as
    long as one of them: one after the other they would take four times.  (The
    runtime deals streams to a few hardware queues, where two may share one:
    the best of several draws.)"""
    import time

    import torch

    require_gpu()
    p = _problem("euler", n, A.TRANSMISSIVE)

    def timed(some):
        best = float("inf")
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for L in some:
                L.step(1024)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        return best

    ratio = []
    for _ in range(4):
        lats = []
        for _ in range(4):
            L = A.Lattice(A.config_from(p, precision=prec), stream=torch.cuda.Stream())
            L.set_state(p.U0)
            lats.append(L)
        one, four = timed(lats[:1]), timed(lats)
        say(f"[grid march] {n} cells prec={prec}: one lattice {1e6 * one:.0f} us, four on streams {1e6 * four:.0f} us")
        ratio.append(four / one)
        for L in lats:
            L.close()
    assert min(ratio) < 3.0, ratio


@pytest.mark.parametrize("prec,sizes", [(A.F32, (14848, 14849, 29697, 59392, 59393)), (A.F64, (14849, 29696, 29697))])
@pytest.mark.parametrize("kind,face", [("advection", A.PERIODIC), ("euler", A.PERIODIC), ("reactive", A.REFLECTIVE)])
def test_bounds_of_many_workgroups(kind, face, prec, sizes):
    """As many workgroups as a wave has lanes, one more, more than the lanes of
    the two waves that hear their bounds, and the last size of the march and
    the first beyond it."""
    require_gpu()
    for n in sizes:
        p = _problem(kind, n, face)
        say(f"[grid march, many workgroups] {kind} face={face} prec={prec} {n} cells")
        a, b = (gpu_lattice(p, prec) for _ in range(2))
        a.step(33)
        for _ in range(33):
            b.step(1)
        assert a.sync(check=False) == b.sync(check=False) and np.array_equal(a.moments(), b.moments()), n
        a.close()
        b.close()


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("n", [929, 4096, 15000])
def test_march_that_is_given_up(n, prec):
    """With no look at what the others wrote every workgroup gives up behind
    its first step: a status and an error of its own, not a non-finite state;
    the steps that were not taken are not steps at the stop time; and a state
    set again is stepped as ever."""
    require_gpu()
    p = _problem("euler", n, A.TRANSMISSIVE)
    say(f"[grid march, given up] {n} cells prec={prec}")
    L = gpu_lattice(p, prec)
    L.step(3)
    L.set_march_limits(hear_looks=0)
    L.step(40)
    st = L.sync(check=False)
    assert st["rc"] == A.EDEVICE and st["flags"] == A.FLAG_STALLED and st["first_bad_step"] == 3, st
    assert st["step"] == 43
    with pytest.raises(A.ArlbmError) as e:
        L.sync()
    assert e.value.code == A.EDEVICE
    assert L.step_until(2.0 * st["t"] + 1.0) == 0  # not stepped on
    L.set_march_limits()
    L.set_state(p.U0)
    ref = gpu_lattice(p, prec)
    L.step(40)
    for _ in range(40):
        ref.step(1)
    assert L.sync() == ref.sync() and np.array_equal(L.moments(), ref.moments())
    L.close()
    ref.close()


def test_state_of_a_given_up_march_in_a_server():
    """A saved state of a march that was given up leaves a server's mix early,
    with the same error."""
    require_gpu()
    p = _problem("euler", 4096, A.TRANSMISSIVE)
    L = gpu_lattice(p, A.F32)
    L.set_march_limits(hear_looks=0)
    L.step(40)
    blob = L.save_state()
    L.close()
    srv = A.Server(1 << 28, A.F32)
    rid = srv.submit_state(A.config_from(p, precision=A.F32), blob, 2000)
    done = []
    for _ in range(4000):
        srv.iterate()
        done = srv.poll(4)
        if done:
            break
    srv.close()
    say("[grid march, given up] served:", done)
    assert done[0]["id"] == rid and done[0]["status"] == A.EDEVICE and done[0]["steps"] < 100
    assert done[0]["flags"] & A.FLAG_STALLED and done[0]["U"] is None


@pytest.mark.parametrize("prec", [A.F32, A.F64])
@pytest.mark.parametrize("kind,n", [("euler", 600), ("euler", 4096), ("swe", 2000), ("reactive", 1000)])
def test_saved_state_holds_the_moments(kind, n, prec):
    """The moment planes of a saved state are the moments of its populations,
    however the steps before it were launched."""
    require_gpu()
    p = _problem(kind, n, A.TRANSMISSIVE)
    a, b = (gpu_lattice(p, prec) for _ in range(2))
    a.step(40)
    for _ in range(40):
        b.step(1)
    real, stride = (np.float32 if prec == A.F32 else np.float64), (n + 63) // 64 * 64 + 1088

    def planes(L):
        blob, f = L.save_state(), int(L.sizes.f_bytes)
        fp = np.frombuffer(blob, dtype=real, count=L.q * L.m * stride, offset=56).reshape(L.q * L.m, stride)[:, :n]
        up = np.frombuffer(blob, dtype=real, count=L.m * stride, offset=56 + f).reshape(L.m, stride)[:, :n]
        return blob[:56], fp, up

    (ha, fa, ua), (hb, fb, ub) = planes(a), planes(b)
    say(f"[saved 1d state] {kind} {n} cells prec={prec}")
    assert ha == hb and np.array_equal(fa, fb) and np.array_equal(ua, ub)
    assert np.array_equal(ua.astype(np.float64), a.moments())
    a.close()
    b.close()
