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
