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
