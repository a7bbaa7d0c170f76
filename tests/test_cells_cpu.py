"""Planning of the cell launches on the CPU."""
import hashlib
import os
import subprocess
import threading
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


def _threads_run_side_by_side():
    """Whether four threads hash (without the interpreter's lock) in less than twice the time of one."""
    data = bytes(32 << 20)

    def took(n):
        th = [threading.Thread(target=lambda: hashlib.sha256(data).digest()) for _ in range(n)]
        t = time.perf_counter()
        for h in th:
            h.start()
        for h in th:
            h.join()
        return time.perf_counter() - t

    return max(took(4) for _ in range(5)) < 1.7 * min(took(1) for _ in range(5))


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
    assert plan(64)[1] < 1.28 * plan(65)[1]  # (but no second copy of the multipliers)
    ratio = []
    for _ in range(8):
        a, b = zip(*((plan(64)[0], plan(65)[0]) for _ in range(4)))
        ratio.append(min(a) / min(b))
        if ratio[-1] < 1.12:
            return
    if not _threads_run_side_by_side():
        pytest.skip("other work keeps this machine's threads from running side by side")
    assert False, ratio


# stage forms (narrow layers, up to four nodes, two-row variables) and kind of the plans that the GPU tests
# of the cells run, so that those tests fail to cover a form only with this one
FORMS = {
    "one_row": (1, 0, 64), "potts1x2_L2": (1, 2, 64), "potts5x7_L3": (1, 0, 512), "potts16x16_L4": (2, 2, 64),
    "potts33x17_L2": (2, 2, 64), "potts40x31_L7": (2, 2, 64), "potts12x9_L16": (2, 2, 64), "star16": (1, 1, 64),
    "star17": (1, 0, 64), "star64": (1, 0, 64), "wide4": (1, 1, 64), "wide4_long": (1, 1, 64), "wide12": (0, 0, 0),
    "tracking200": (1, 0, 64), "tracking1400": (1, 1, 256), "tracking1800": (2, 1, 128), "tracking_batch": (1, 1, 256),
    "potts_and_tracking": (2, 1, 512),
}


@pytest.mark.parametrize("name", sorted(FORMS))
def test_cell_forms_of_the_gpu_cases(name):
    from test_gpu_cells import CASES

    assert set(FORMS) == set(CASES)
    probs = [B.Problem.from_ilp(q) for q in CASES[name]()]
    c = B.Plan(probs if len(probs) > 1 else probs[0], hist_cap=64).cells()
    kind, form, lanes = FORMS[name]
    assert (c["kind"], c["form"][1], c["lanes"][1]) == (kind, form, lanes)
    assert (c["n_cells"][0] > 0) == (kind == 2) and (c["n_cells"][1] > 0) == (kind > 0)
    assert all(q <= 160 << 10 for q in c["lds"])


def test_plans_without_cells_say_so():
    """Splits, levels of more than four nodes and variables in more than 64 rows have none."""
    grid = B.Problem.from_ilp(I.potts_grid(4, 4, 2, seed=1))
    for plan in (B.Plan(grid, n_intervals=2), B.Plan(B.Problem.from_ilp(I.tomography(16))),
                 B.Plan(B.Problem.from_ilp(star(65, 2, 1)))):
        assert plan.cells() == dict(kind=0, from_=0, n_cells=(0, 0), form=(0, 0), lanes=(0, 0), lds=(0, 0))
    assert B.Plan(grid).cells()["kind"] == 1


def test_quotient_by_a_row_count(tmp_path):
    """The cells' division by a variable's number of rows is correctly rounded: every mantissa over 1 to 64,
    both signs, at the ends of the range that takes the correction and beyond it."""
    src = tmp_path / "q.cpp"
    src.write_text("""
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include "quotient.h"
static int bad = 0;
static void check(float s, float n, float r) {
  const float a = bddmp::over_count(s, n, r), b = s / n;
  if (std::memcmp(&a, &b, 4) && bad++ < 5) std::printf("%a / %g: %a, not %a\\n", s, n, a, b);
}
int main() {
  for (int n = 1; n <= 64; ++n) {
    const float r = 1.0f / float(n);
    for (int m = 0; m < 1 << 23; ++m) check(std::ldexp(1.0f + m * 0x1p-23f, m & 1 ? 3 : -40), float(n), r);
    for (int e = -149; e < 128; ++e)
      for (int m = 0; m < 1 << 23; m += 104729)
        for (float sign : {1.0f, -1.0f}) check(sign * std::ldexp(1.0f + m * 0x1p-23f, e), float(n), r);
    for (float s : {0.0f, INFINITY, -INFINITY}) check(s, float(n), r);
  }
  return bad != 0;
}
""")
    exe = str(tmp_path / "q")
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=off", "-std=c++17", "-I",
                    os.path.join(os.path.dirname(B.LIB_PATH), "csrc"), str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


def random_rows(n, m, k, cmax=1, rhs=1, seed=1):
    """m rows of k variables, one from each of k blocks of the order."""
    r = np.random.default_rng([n, m, k, seed])
    col = (r.integers(0, n // k, (m, k)) + np.arange(k) * (n // k)).reshape(-1)
    coef = r.integers(1, cmax + 1, (16, k))[r.integers(0, 16, m)].reshape(-1)
    return I.ILP(n, r.standard_normal(n), np.arange(m + 1) * k, col.astype(np.int32), coef, np.ones(m, np.int8),
                 np.full(m, rhs, np.int64), None)


@pytest.mark.parametrize("make,count,kind,short", [
    # one component of many layers in few steps keeps a compute unit busy alone
    (lambda s: random_rows(900, 2300, 2, seed=s), 40, 0, False),
    (lambda s: random_rows(1500, 1700, 3, 2, 3, seed=s), 300, 0, False),
    (lambda s: random_rows(1500, 1700, 3, 2, 3, seed=s), 1, 1, True),
    (lambda s: random_rows(1600, 600, 8, seed=s), 1, 1, False),
    (lambda s: random_rows(1600, 600, 8, 2, 3, seed=s), 64, 1, False),
    # two stages that hand every message on to another place
    (lambda s: random_rows(100000, 100000, 2, seed=s), 1, 0, False),
    (lambda s: I.potts_grid(300, 300, 2, seed=s), 1, 2, True),
    (lambda s: I.potts_grid(128, 128, 4, seed=s), 1, 2, False),
    (lambda s: I.tracking(300, seed=s), 8, 1, False),
])
def test_cells_run_where_they_take_less_time(make, count, kind, short):
    """Few large components of few steps, and scattered boundaries, took up to 1.9 times as long as cells; calls
    of few iterations pay for gathering the multipliers."""
    q = [B.Problem.from_ilp(p, order=p.order is not None) for p in (make(s) for s in range(count))]
    c = B.Plan(q if count > 1 else q[0], hist_cap=64).cells()
    assert c["kind"] == kind
    assert (c["from_"] > 1) == short and (c["from_"] > 0) == (kind > 0)
