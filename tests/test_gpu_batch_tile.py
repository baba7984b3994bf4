"""Several steps of every plane of a batch in one launch: bit for bit the single steps of the XCD-placed
order, which are never taken together.

The batches mix planes that fit in a work-group (from one cell, one row, one column on) with planes that need
several, with last tiles of a row or two, at few and at many domains, so that the rule takes both sizes of
work-group and several numbers of steps; steps in calls of less than, exactly and more than a launch.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lbm = pytest.importorskip("paper_2605_27004_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("storage,count,lo,hi,order", [
    ("f32", 0, 0, 0, 3), ("f64", 0, 0, 0, 2), ("f32", 4, 10, 22, 3), ("f64", 60, 10, 40, 3), ("f32", 128, 30, 64, 2),
    ("f64", 300, 16, 64, 3), ("f32", 2, 60, 150, 3)])
def test_launch_of_several_steps_is_single_steps(storage, count, lo, hi, order):
    rng = np.random.default_rng(29)
    edges = [(1, 1), (1, 30), (30, 1), (2, 2), (3, 170), (16, 32), (17, 31), (32, 32), (33, 32), (64, 16), (64, 17),
             (23, 45), (64, 64)]
    edges += [tuple(int(v) for v in rng.integers(lo, hi + 1, 2)) for _ in range(count)]
    doms = []
    for i, (nx, ny) in enumerate(edges):
        rho, s = W.random_fields((nx, ny, 1), 2, 200 + i)
        doms.append(dict(shape=(nx, ny, 1), tensor=W.config1_theta(), tensor_kind="theta",
                         tau=float(rng.uniform(0.6, 1.4)), rho=rho, s=s))
    b = lbm.Batch("D2Q9", storage, doms, order=order)
    c = lbm.Batch("D2Q9", storage, doms, order=order)
    c.set_schedule(mode="stepwise", xcd_group=1)
    for k in (1, 37, 2, 16, 5):
        b.step(k)
        c.step(k)
        assert b.t == c.t
        assert torch.equal(b.f64(), c.f64())
    b.close()
    c.close()
