"""Planning of the cell launches on the CPU."""
import os
import time

import numpy as np
import pytest

from paper_2009_00481_amd import binding as B
from paper_2009_00481_amd import instances as I


def star(m, k, seed):
    """m rows sharing variable 0, each with k variables of its own (cells take up to 64 rows a variable)."""
    rng = np.random.default_rng(seed)
    rows = [(np.concatenate([[0], 1 + j * k + np.arange(k)]), np.ones(k + 1, int), 1, 1) for j in range(m)]
    n = 1 + m * k
    return I.from_rows(n, rng.standard_normal(n), rows)


@pytest.mark.skipif(len(os.sched_getaffinity(0)) < 4, reason="the cells are planned on threads beside the rest")
def test_cells_cost_a_plan_little_time():
    """A plan with cells against the same plan without (one variable in 65 rows): the cells' planning was up
    to 1.4 times a plan's time. The least of several tries, so that other work on the machine does not decide."""
    def plan(rows):
        q = [B.Problem.from_ilp(I.potts_grid(64, 64, 4, seed=1)), B.Problem.from_ilp(star(rows, 2, 2))]
        t = time.perf_counter()
        p = B.Plan(q, hist_cap=64)
        return time.perf_counter() - t, int(p.stats.device_bytes)

    assert plan(64)[1] > 1.2 * plan(65)[1]  # (the one with cells holds their arrays)
    ratio = []
    for _ in range(8):
        a, b = zip(*((plan(64)[0], plan(65)[0]) for _ in range(4)))
        ratio.append(min(a) / min(b))
        if ratio[-1] < 1.12:
            return
    assert False, ratio
