"""The pinned places that read-outs take: a call that fails after a kernel which writes to its place was enqueued
must not give that place to the next call before the stream has been waited for. (No GPU: the launches are
listed, and fail on request.)"""
from tests import fake_hip


def test_place_of_a_failed_gradient_is_not_given_away():
    out = fake_hip.run("""
c = make("D3Q19", "f32", (16, 16, 16))
d = make("D3Q19", "f32", (16, 16, 16))
spec = lbm.make_grad_spec("kinetic_energy", 3, 3)
out = {}
lbm.lbm_objective(d)
out["first"] = [l["args"][3] for l in fake.launches() if "k_sum" in l["name"]]
for waits in (True, False):
    fake.fail("k_adjoint", 1)
    fake.capture(not waits)       # a stream that cannot be waited for
    try:
        lbm.lbm_grad(c, spec, 1 << 50)
        raise SystemExit("the gradient should have failed")
    except lbm.LBMError as e:
        assert e.code == lbm.LBM_ERR_HIP
    failed = [l["args"][3] for l in fake.launches() if "k_sum" in l["name"]]
    fake.capture(False)
    fake.fail("")
    lbm.lbm_objective(d)
    out[str(waits)] = [failed, [l["args"][3] for l in fake.launches() if "k_sum" in l["name"]]]
""")
    # after a wait the place is free again; without one it stays with the kernel that may write to it
    assert out["True"] == [out["first"], out["first"]]
    failed, nxt = out["False"]
    assert failed == out["first"] and nxt != failed


def test_totals_without_a_place():
    """Sixteen calls that cannot wait use all places up; the next calls copy, from the scratch."""
    out = fake_hip.run("""
c = make("D3Q19", "f32", (16, 16, 16))
fake.capture(True)
for i in range(16):
    try:
        lbm.lbm_moments(c, None, None, True)
        raise SystemExit("a stream that is being recorded cannot be waited for")
    except lbm.LBMError:
        pass
fake.launches()
fake.capture(False)
tot = lbm.lbm_moments(c, None, None, True)
to = [l["args"][2] for l in fake.launches() if "k_reduce" in l["name"]][0]
b = make_batch("D2Q9", "f64", [(4, 4, 1)] * 3)
rows = lbm.lbm_batch_moments(b, None, None, 3)
out = dict(tot=tot, scratch=SCRATCH <= to < RHO, rows=len(rows))
""")
    # (the stand-in's copies read zeros: no fluid cells in the grid, rho0 times the cells in the batch)
    assert out == dict(tot=[0.0, 0.0, 0.0, 0.0], scratch=True, rows=3)
