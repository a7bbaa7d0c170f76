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
