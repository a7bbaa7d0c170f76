"""The solver's host code on a HIP runtime without a device: which copies it checks and which kernels it
launches. No kernel runs."""
import pytest

import hip_stub


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return hip_stub.build(tmp_path_factory.mktemp("hip"))


@pytest.mark.parametrize("plan", ["I.config('5sub')", "I.tomography(8)", "I.tracking(300, seed=1)"])
def test_bind_fails_when_any_upload_fails(stub, plan):
    """A plan array that did not arrive would hold whatever the arena held, which the kernels index with."""
    out = hip_stub.run(stub, f"""
plan = B.Plan(B.Problem.from_ilp({plan}))
stub.stub_fail_upload(-1)
bind(plan)
n = stub.stub_uploads()
missed = []
for k in range(n):
    stub.stub_fail_upload(k)
    launches()
    try:
        bind(plan)
        missed.append(k)
    except B.BddmpError as e:
        assert e.code == -6, e
        if launches():
            missed.append(k)
print(n, missed)
""")
    n, missed = out.split(None, 1)
    assert int(n) > 20
    assert missed.strip() == "[]"


@pytest.mark.parametrize("launch", [(0, 0), (3, 4)])
def test_autotune_times_the_paths_it_chooses_between(stub, launch):
    """Cells have no general-layer path: a plan that runs as cells is tuned on its wave launches, or on the
    selected form's, and runs as cells again afterwards."""
    out = hip_stub.run(stub, f"""
plan = B.Plan(B.Problem.from_ilp(I.tracking(1400, seed=1)))
h = bind(plan)
if {launch[0]}:
    B.bddmp_solver_set_launch(h, *{launch})
launches()
B.bddmp_solver_autotune(h, 2)
tuned = launches()
B.bddmp_solver_iterate(h, 2)
after = launches()
for name in (tuned, after):
    print(*(sum(k in q for q in name) for k in ("cell_kernel", "wave_kernel", "group_kernel")))
""")
    tuned, after = ([int(v) for v in line.split()] for line in out.splitlines())
    assert tuned[0] == 0 and max(tuned[1:]) > 0
    assert (after[0] > 0) == (launch[0] == 0)


@pytest.mark.parametrize("kib,cells", [(160, True), (64, False)])
def test_cells_run_where_the_device_holds_them(stub, kib, cells):
    """A cell of this plan takes 138 KB of LDS: on a device with less to a workgroup the iterations run as
    wave launches, as they do without cells."""
    out = hip_stub.run(stub, f"""
plan = B.Plan(B.Problem.from_ilp(I.tracking(1400, seed=1)))
stub.stub_set_lds({kib} << 10)
h = bind(plan)
launches()
B.bddmp_solver_iterate(h, 3)
names = launches()
print(*(sum(k in q for q in names) for k in ("cell_kernel", "wave_kernel")))
# (a plan whose cells are small)
small = B.Plan(B.Problem.from_ilp(I.potts_grid(3, 3, 2, seed=1)))
h = bind(small)
launches()
B.bddmp_solver_iterate(h, 3)
print(sum("cell_kernel" in q for q in launches()))
""").split()
    assert (int(out[0]) > 0) == cells and (int(out[1]) > 0) == (not cells)
    assert int(out[2]) > 0


# random rows of k variables, one from each of k blocks of the order: k waves, layers that lie apart
RANDOM_ROWS = """
def random_rows(m, k, cmax=1, rhs=1):
    r = np.random.default_rng([m, k])
    n = m * k
    col = (r.integers(0, m, (m, k)) + np.arange(k) * m).reshape(-1)
    coef = r.integers(1, cmax + 1, (16, k))[r.integers(0, 16, m)].reshape(-1)
    return I.ILP(n, r.standard_normal(n), np.arange(m + 1) * k, col.astype(np.int32), coef, np.ones(m, np.int8),
                 np.full(m, rhs, np.int64), None)
"""


@pytest.mark.parametrize("plan,rows", [
    ("random_rows(25000, 2)", True),
    ("random_rows(200000, 2)", False),
    ("random_rows(50000, 8)", True),
    ("random_rows(200000, 8)", False),
    ("I.potts_grid(96, 96, 4, seed=1)", True),
    ("random_rows(8000, 5, 3, 3)", True),
    ("random_rows(60000, 5, 3, 3)", False),
    ("I.tomography(16)", True),
])
def test_passes_without_updates_run_by_rows_where_that_is_faster(stub, plan, rows):
    """Few waves of many layers that lie apart, or of many short rows of wide levels, take a launch per wave:
    by rows they took up to 2.7 times as long."""
    out = hip_stub.run(stub, RANDOM_ROWS + f"""
plan = B.Plan(B.Problem.from_ilp({plan}, order=False))
h = bind(plan)
launches()
B.bddmp_solver_reset(h)
a = launches()
B._check(L.bddmp_solver_min_marginals(h, None, None))
b = launches()
for name in (a, b):
    print(*(sum(k in q for q in name) for k in ("wave_kernel", "row_")))
""").split()
    assert [int(v) > 0 for v in out] == [not rows, rows] * 2


def test_short_calls_run_without_cells(stub):
    """Where gathering the multipliers costs more than a few iterations gain, short calls are replays."""
    out = hip_stub.run(stub, """
plan = B.Plan(B.Problem.from_ilp(I.potts_grid(300, 300, 2, seed=1)))
k = plan.cells()["from_"]
h = bind(plan)
print(k)
for n in (1, k - 1, k, k + 1, 1):
    launches()
    B.bddmp_solver_iterate(h, n)
    names = launches()
    print(*(sum(q in x for x in names) > 0 for q in ("cell_kernel", "wave_kernel")))
""").splitlines()
    assert int(out[0]) > 1
    assert out[1:] == ["False True", "False True", "True False", "True False", "False True"]
