"""GPU tests of the wave kernels' tiles at the edges of their forms, bitwise against the oracle's float
mirror: the exchange sum of variables in few to many rows (blocks of eight and four rows, a workgroup's
tile and more), rows that force the variable among them, tiles of general levels at the sizes where
their node maps end, and the passes that run by rows."""
import numpy as np
import pytest

from oracle import Oracle
from paper_2009_00481_amd import binding as B
from paper_2009_00481_amd import instances as I

pytestmark = pytest.mark.gpu


def _check(ilp, T, **opt):
    plan = B.Plan(B.Problem.from_ilp(ilp), **opt)
    s = B.Solver(plan)
    s.set_graphs(False)
    s.iterate(T)
    m0, m1 = s.min_marginals()
    o = Oracle(I.ILP(ilp.n, ilp.cost, ilp.row_ptr, ilp.col, ilp.coef, ilp.sense, ilp.rhs, plan.order()), precision="f32")
    o.init()
    o.iterate(T)
    r0, r1 = o.min_marginals()
    for got, want in ((s.get_lambda(), o.lam()), (m0, r0), (m1, r1)):
        assert np.array_equal(got.cpu().numpy().astype(np.float64), np.asarray(want, np.float64))


@pytest.mark.parametrize("forced", [0, 3])
@pytest.mark.parametrize("m", [1, 3, 4, 5, 7, 8, 9, 12, 13, 45, 64, 65, 200, 256, 257, 300])
def test_exchange_sums_bitwise(m, forced):
    """m rows share variable 0; forced of them more hold it at 0 (one-variable rows: infinite differences)."""
    rng = np.random.default_rng([m, forced])
    rows = []
    for j in range(m):
        v = np.array([0, 1 + 2 * j, 2 + 2 * j])
        rows.append((v, rng.choice([-1, 1], 3), int(rng.integers(1, 3)), 0))
    for j in range(forced):
        rows.insert(int(rng.integers(0, len(rows) + 1)), (np.array([0]), np.array([1]), 1, 0))
    n = 1 + 2 * m
    _check(I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows), 3)


@pytest.mark.parametrize("m,k,cmax,rhs", [(255, 5, 3, 7), (256, 5, 3, 7), (257, 5, 3, 7), (600, 4, 2, 4), (40, 9, 40, 120),
                                          (9, 14, 300, 1500), (1, 12, 5, 20)])
@pytest.mark.parametrize("work", [0, 2048, 100000])
def test_general_tiles_bitwise(m, k, cmax, rhs, work):
    """m rows over variables of their own: every wave holds one level of each row."""
    rng = np.random.default_rng([m, k, cmax])
    rows = [(np.arange(j * k, (j + 1) * k), rng.integers(1, cmax + 1, k), 1, rhs) for j in range(m)]
    n = m * k
    _check(I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows), 2, tile_work=work)


@pytest.mark.parametrize("k", [1, 2, 7, 8, 9, 15, 16, 17, 40])
@pytest.mark.parametrize("m", [1, 255, 257])
def test_row_passes_bitwise(m, k):
    """Initial sweep from given multipliers and min-marginals by rows, at the edges of their blocks of eight
    levels and of a workgroup's rows; m rows of k to k + 2 levels, each sharing a variable with the next."""
    rng = np.random.default_rng([m, k])
    rows, v = [], 0
    for j in range(m):
        kk = k + j % 3 if k > 1 else 1
        rows.append((np.arange(v, v + kk), np.ones(kk, int), j % 2, 1))
        v += max(kk - 1, 1)
    n = v + 2
    ilp = I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows)
    plan = B.Plan(B.Problem.from_ilp(ilp))
    lam = rng.standard_normal(int(plan.stats.n_incidences)).astype(np.float32)
    import torch

    s = B.Solver(plan)
    s.set_lambda(torch.from_numpy(lam).cuda())
    o = Oracle(I.ILP(ilp.n, ilp.cost, ilp.row_ptr, ilp.col, ilp.coef, ilp.sense, ilp.rhs, plan.order()), precision="f32")
    o.init()
    o.set_lambda(lam.astype(np.float64))
    for step in range(2):
        m0, m1 = s.min_marginals()
        r0, r1 = o.min_marginals()
        assert np.array_equal(m0.cpu().numpy().astype(np.float64), r0) and np.array_equal(m1.cpu().numpy().astype(np.float64), r1)
        np.testing.assert_allclose(s.lb_history(1)[-1], o.lower_bound(), rtol=1e-12, atol=1e-9)
        s.iterate(1)
        o.iterate(1)


@pytest.mark.parametrize("k,cmax,rhs", [(1, 2, 2), (6, 5, 9), (63, 3, 40), (64, 3, 40), (65, 3, 40), (130, 2, 70), (16, 200, 900)])
@pytest.mark.parametrize("m", [1, 5])
def test_wide_row_passes_bitwise(m, k, cmax, rhs):
    """The same with levels of more than two nodes (up to some hundreds): one row per wavefront, 64 levels'
    records at a time, more nodes than lanes."""
    import torch

    rng = np.random.default_rng([m, k, cmax])
    rows = [(np.arange(j * (k - 1), j * (k - 1) + k) if k > 1 else np.array([j]), rng.integers(1, cmax + 1, k), 1, rhs)
            for j in range(m)]
    n = m * max(k - 1, 1) + 1
    ilp = I.from_rows(n, rng.standard_normal(n, dtype=np.float32).astype(np.float64), rows)
    plan = B.Plan(B.Problem.from_ilp(ilp))
    lam = rng.standard_normal(int(plan.stats.n_incidences)).astype(np.float32)
    s = B.Solver(plan)
    s.set_lambda(torch.from_numpy(lam).cuda())
    o = Oracle(I.ILP(ilp.n, ilp.cost, ilp.row_ptr, ilp.col, ilp.coef, ilp.sense, ilp.rhs, plan.order()), precision="f32")
    o.init()
    o.set_lambda(lam.astype(np.float64))
    for step in range(2):
        m0, m1 = s.min_marginals()
        r0, r1 = o.min_marginals()
        assert np.array_equal(m0.cpu().numpy().astype(np.float64), r0) and np.array_equal(m1.cpu().numpy().astype(np.float64), r1)
        np.testing.assert_allclose(s.lb_history(1)[-1], o.lower_bound(), rtol=1e-12, atol=1e-9)
        s.iterate(1)
        o.iterate(1)
