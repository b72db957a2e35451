"""Launches of a time-targeted run (arlbm_step_until): a saved state's header
counts them, those that took no step among them."""
import math
import struct

import numpy as np
import pytest

from paper_2609_18177_amd import arlbm as A
from paper_2609_18177_amd import workloads as W
from gpu_common import gpu_lattice, require_gpu, say
from helpers import ora_from

pytestmark = pytest.mark.gpu


def _blast(dim, n):
    """One cell at ten times the pressure around it: the time step grows
    threefold while the blast spreads over its first cells."""
    p = W.euler_seeded_2d(0, n=n) if dim == 2 else W.euler_octants_3d(seed=0, n=n)
    shape = (n,) * dim
    pr = np.ones(shape)
    pr[(n // 2,) * dim] = 10.0
    p.U0 = np.stack([np.ones(shape)] + [np.zeros(shape)] * dim + [pr / 0.4])
    return p


@pytest.mark.parametrize("dim,n,steps", [(2, 96, 300), (3, 20, 60)])
def test_surplus_launches_of_a_growing_time_step(dim, n, steps):
    """A run whose launches each take a step is sized by a trial step: it makes
    no more of them than two launches and then, as often as it takes, the
    time left over the last time step and one."""
    require_gpu()
    p = _blast(dim, n)
    Lo = ora_from(p)
    dts, t = [], 0.0
    for _ in range(steps + 2):
        Lo.run(1)
        dts.append(Lo.t - t)
        t = Lo.t
    goal = sum(dts[:steps]) - 0.5 * dts[steps - 1]
    t, done, allowed, last = 0.0, 0, 0, 0.0
    while t < goal:
        k = 2 if done == 0 else math.ceil((goal - t) / last) + 1
        allowed += k
        for _ in range(k):
            if t < goal:
                last, t, done = dts[done], t + dts[done], done + 1
    G = gpu_lattice(p, A.F64)
    taken = G.step_until(goal)
    launches = struct.unpack_from("<q", G.save_state(), 32)[0]
    G.close()
    say(f"[until] {dim}D blast {n} cells a side: {taken} steps, {launches} launches, at most {allowed}")
    assert taken == done == steps
    assert launches <= allowed + 1
