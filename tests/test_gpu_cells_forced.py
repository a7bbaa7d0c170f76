"""GPU tests of the cell kernels where rows force variables (one-variable rows: infinite differences), in
each form of cells and through each branch of the exchange: bitwise against host-launched waves and the
oracle's float mirror."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2009_00481_amd import binding as B
from paper_2009_00481_amd import instances as I

pytestmark = pytest.mark.gpu

LAYERS, UP_TO_FOUR, PAIRS = 0, 1, 2  # forms of bddmp_cells


def _chain(n, seed):
    """x_j + x_{j+1} <= 1 along n variables, each in two rows: the ends' second rows fix them at 0 and 1."""
    rng = np.random.default_rng([n, seed])
    rows = [(np.array([j, j + 1]), np.array([1, 1]), 1, 1) for j in range(n - 1)]
    rows.insert(int(rng.integers(0, n)), (np.array([0]), np.array([1]), 1, 0))
    rows.insert(int(rng.integers(0, n)), (np.array([n - 1]), np.array([1]), 2, 1))
    return I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows)


def _doubly_fixed(n, seed):
    """n variables in two rows each: every third with both rows fixing it, the others with one."""
    rng = np.random.default_rng([n, seed])
    rows = []
    for j in range(0, n, 3):
        k = min(3, n - j)
        rows += [(np.array([j]), np.array([1]), j % 2 + 1, j % 2)] * 2  # <= 0 or >= 1, twice
        if k > 1:
            rows.append((np.arange(j + 1, j + k), np.ones(k - 1, int), 1, 1))
            rows += [(np.array([q]), np.array([1]), 1, 0) for q in range(j + 1, j + k)]
    return I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows)


def _star(m, forced, cmax, at, seed):
    """m rows share variable 0 with k more variables each; forced of the rows hold it at ``at``."""
    rng = np.random.default_rng([m, forced, cmax, seed])
    rows, k = [], 2 * cmax
    for j in range(m - forced):
        v = np.concatenate([[0], 1 + k * j + np.arange(k)])
        if cmax > 1:
            rows.append((v, rng.integers(1, cmax + 1, k + 1), 1, 3))
        else:
            rows.append((v, np.ones(k + 1, int), 1, 1))
    for j in range(forced):
        rows.insert(int(rng.integers(0, len(rows) + 1)), (np.array([0]), np.array([1]), 1 + at, at))
    n = 1 + k * (m - forced)
    return I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows)


def _grid(h, w, fixed, seed):
    """Pairs of neighbours on a grid exclude each other (variables in two to four rows); some fixed at 0."""
    rng = np.random.default_rng([h, w, seed])
    at = np.arange(h * w).reshape(h, w)
    rows = [(np.array(p), np.array([1, 1]), 1, 1) for p in [*zip(at[:, :-1].flat, at[:, 1:].flat),
                                                           *zip(at[:-1].flat, at[1:].flat)]]
    rows += [(np.array([q]), np.array([1]), 1, 0) for q in rng.choice(h * w, fixed, replace=False)]
    return I.from_rows(h * w, rng.standard_normal(h * w, dtype=np.float32).astype(np.float64),
                       [rows[q] for q in rng.permutation(len(rows))])


def _bipartite(n, m, fixed, seed):
    """Rows over a variable of either half of the order: two steps of many variables (several wavefronts)."""
    rng = np.random.default_rng([n, m, seed])
    pairs = {(int(a), int(b)) for a, b in zip(rng.integers(0, n // 2, m), rng.integers(n // 2, n, m))}
    rows = [(np.array(p), np.array([1, 1]), 1, 1) for p in sorted(pairs)]
    rows += [(np.array([q]), np.array([1]), 1, 0) for q in rng.choice(n, fixed, replace=False)]
    return I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64),
                       [rows[q] for q in rng.permutation(len(rows))])


CASES = {f"chain{n}": (lambda n=n: _chain(n, 1), PAIRS) for n in (2, 3, 33, 64, 65, 500, 2000)}
CASES.update({f"fixed{n}": (lambda n=n: _doubly_fixed(n, 2), PAIRS) for n in (1, 3, 5, 200, 1000)})
CASES.update({f"grid{h}x{w}": (lambda h=h, w=w: _grid(h, w, 1 + h * w // 7, 5), LAYERS)
              for h, w in ((2, 3), (9, 9), (20, 20), (5, 200), (1, 1000))})
CASES.update({f"bipartite{n}_{m}": (lambda n=n, m=m: _bipartite(n, m, n // 9, 6), LAYERS) for n, m in ((300, 450), (150, 900))})
# few rows (sums by register moves), up to 16 (handed from lane to lane), more (lane reads)
for _m in (2, 3, 15, 16, 17, 64):
    for _f in (1, 2):
        for _at in (0, 1):
            if _f < _m:
                CASES[f"star{_m}_{_f}_at{_at}"] = (lambda m=_m, f=_f, at=_at: _star(m, f, 1, at, 3), LAYERS)
                CASES[f"wide{_m}_{_f}_at{_at}"] = (lambda m=_m, f=_f, at=_at: _star(m, f, 2, at, 4), UP_TO_FOUR)


@pytest.mark.parametrize("name", sorted(CASES))
def test_forced_rows_in_cells_bitwise(name):
    make, form = CASES[name]
    ilp = make()
    plan = B.Plan(B.Problem.from_ilp(ilp), hist_cap=64)
    cells = plan.cells()
    assert cells["kind"] > 0 and cells["form"][1] == form
    assert not name.startswith("bipartite") or cells["lanes"][1] > 64
    out = []
    for graphs in (True, False):
        s = B.Solver(plan)
        s.set_graphs(graphs)
        for n in (1, 4):
            s.iterate(n)
        m0, m1 = s.min_marginals()
        out.append([s.get_lambda().cpu().numpy(), m0.cpu().numpy(), m1.cpu().numpy(), s.lb_history(64)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    o = Oracle(I.ILP(ilp.n, ilp.cost, ilp.row_ptr, ilp.col, ilp.coef, ilp.sense, ilp.rhs, plan.order()), precision="f32")
    o.init()
    o.iterate(5)
    r0, r1 = o.min_marginals()
    for got, want in zip(out[0], (o.lam(), r0, r1)):
        assert np.array_equal(got.astype(np.float64), np.asarray(want, np.float64))
    # (the variables of these rows are forced: differences are infinite)
    assert np.isinf(r1 - r0).any()


def test_short_calls_between_cells_bitwise():
    """Calls of fewer iterations than cells take run as replayed waves: any sequence gives the same."""
    plan = B.Plan(B.Problem.from_ilp(I.potts_grid(300, 300, 2, seed=1)), hist_cap=64)
    k = plan.cells()["from_"]
    assert plan.cells()["kind"] == 2 and k > 1
    out = []
    for graphs in (True, False):
        s = B.Solver(plan)
        s.set_graphs(graphs)
        for n in (1, k, 1, k - 1, k + 9, 1):
            s.iterate(n)
        m0, m1 = s.min_marginals()
        out.append([v.cpu().numpy() for v in (s.get_lambda(), m0, m1)] + [s.lb_history(64)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
