"""GPU tests of the cell launches (the default launch form's iterations where the plan's components fit
a workgroup): multipliers, bounds, min-marginals, per-instance bounds and every later call bitwise
equal to host-launched waves, at the edges of the cells' forms: one stage and two, one-wavefront and
large cells, two-row variables and others, variables in up to 64 rows, levels of up to 4 nodes (wider
ones run as waves), rings
of bound terms longer and shorter than the run."""
import numpy as np
import pytest

from paper_2009_00481_amd import binding as B
from paper_2009_00481_amd import instances as I

pytestmark = pytest.mark.gpu


def _star(m, k, seed):
    """m rows sharing variable 0, each with k variables of its own: one variable in m rows."""
    rng = np.random.default_rng(seed)
    rows = []
    for j in range(m):
        v = np.concatenate([[0], 1 + j * k + np.arange(k)])
        rows.append((v, rng.choice([-1, 1], v.size), int(rng.integers(1, 3)), 0))
    n = 1 + m * k
    return I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows)


def _wide(m, k, most, seed):
    """Chains of knapsack rows with coefficients up to 3 (levels of up to most + 1 nodes)."""
    rng = np.random.default_rng(seed)
    n = m * (k - 1) + 1
    rows = [(np.arange(j * (k - 1), j * (k - 1) + k), rng.integers(1, 4, k), 1, most) for j in range(m)]
    return I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows)


CASES = {
    "one_row": lambda: [I.from_rows(3, np.array([1.0, -2.0, 0.5]), [([0, 1, 2], [1, 1, 1], 0, 1)])],
    "potts1x2_L2": lambda: [I.potts_grid(1, 2, 2, seed=1)],
    "potts5x7_L3": lambda: [I.potts_grid(5, 7, 3, seed=2)],
    "potts16x16_L4": lambda: [I.config("5sub")],
    "potts33x17_L2": lambda: [I.potts_grid(33, 17, 2, seed=3)],
    "potts40x31_L7": lambda: [I.potts_grid(40, 31, 7, seed=4)],
    "potts12x9_L16": lambda: [I.potts_grid(12, 9, 16, seed=5)],
    "star16": lambda: [_star(16, 3, 6)],
    "star17": lambda: [_star(17, 2, 7)],
    "star64": lambda: [_star(64, 2, 8)],
    "wide4": lambda: [_wide(40, 5, 3, 9)],
    "wide4_long": lambda: [_wide(6, 300, 3, 12)],
    "wide12": lambda: [_wide(40, 9, 11, 9)],
    "tracking200": lambda: [I.tracking(200, seed=10)],
    "tracking1400": lambda: [I.tracking(1400, seed=11)],
    "tracking1800": lambda: [I.tracking(1800, seed=13)],
    "tracking_batch": lambda: [I.tracking(200 + 150 * k, seed=k) for k in range(6)],
    "potts_and_tracking": lambda: [I.potts_grid(20, 30, 4, seed=1), I.tracking(300, seed=2), I.config(1)],
}


def _run(plan, graphs):
    s = B.Solver(plan)
    s.set_graphs(graphs)
    out = []
    for n in (1, 2, 7):
        s.iterate(n)
        out.append(s.get_lambda().cpu().numpy())
    out += [m.cpu().numpy() for m in s.min_marginals()]
    M, x, obj, nv = s.round_primal()
    out += [M.cpu().numpy(), x, np.array([obj, nv]), s.instance_bounds(), s.lb_history(64)]
    # another launch form after cells, and cells after another form and after given multipliers
    s.set_launch(3, 4)
    s.iterate(2)
    s.set_launch(0)
    s.iterate(1)
    s.set_lambda(s.get_lambda().mul_(0.5))
    s.iterate(3)
    out += [s.get_lambda().cpu().numpy(), s.lb_history(64), np.array(s.lower_bound())]
    return out


@pytest.mark.parametrize("name", sorted(CASES))
def test_cells_equal_wave_launches_bitwise(name):
    probs = [B.Problem.from_ilp(q) for q in CASES[name]()]
    plan = B.Plan(probs if len(probs) > 1 else probs[0], hist_cap=64)
    a, b = _run(plan, True), _run(plan, False)
    for k, (x, y) in enumerate(zip(a, b)):
        assert np.array_equal(x, y), (name, k)


@pytest.mark.parametrize("hist_cap", [1, 5, 256])
def test_bound_terms_ring(hist_cap):
    """Runs longer than the ring of bound terms and than the history keep the last bounds."""
    plan = B.Plan(B.Problem.from_ilp(I.potts_grid(6, 5, 3, seed=3)), hist_cap=hist_cap)
    ref = B.Plan(B.Problem.from_ilp(I.potts_grid(6, 5, 3, seed=3)), hist_cap=512)
    s, r = B.Solver(plan), B.Solver(ref)
    r.set_graphs(False)
    s.iterate(150)
    r.iterate(150)
    k = min(hist_cap, 151)
    assert np.array_equal(s.lb_history(k), r.lb_history(151)[-k:])
    assert np.array_equal(s.get_lambda().cpu().numpy(), r.get_lambda().cpu().numpy())
