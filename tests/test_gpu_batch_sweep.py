"""Two steps of every domain of a batch in one launch: bit for bit the single steps of the XCD-placed
order, which are never taken two at a time.

Each batch mixes boxes of the workload's kind, enough of them for the rule to pick the two-step launch,
with the edges of its tiles: extents of 1 to 3, rows of the longest kind, whole cross-sections in one
tile and just too large for it, and more z-planes than a record takes.
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


@pytest.mark.parametrize("lattice,storage,count,order,steps", [
    ("D3Q19", "f32", 60, 3, 7), ("D3Q19", "f64", 40, 2, 5), ("D3Q27", "f32", 60, 2, 5), ("D3Q27", "f64", 50, 3, 7)])
def test_two_step_launch_is_two_steps(lattice, storage, count, order, steps):
    rng = np.random.default_rng(23)
    edges = [(1, 1, 1), (2, 3, 2), (3, 2, 90), (1, 200, 3), (100, 9, 5), (32, 32, 20), (33, 32, 7), (24, 27, 9),
             (20, 21, 70), (64, 16, 3), (63, 10, 4)]
    edges += [tuple(int(v) for v in rng.integers(16, 65, 3)) for _ in range(count)]
    doms = []
    for i, shape in enumerate(edges):
        rho, s = W.random_fields(shape, 3, 100 + i)
        doms.append(dict(shape=shape, tensor=W.random_theta(100 + i), tensor_kind="theta",
                         tau=float(rng.uniform(0.6, 1.4)), rho=rho, s=s))
    b = lbm.Batch(lattice, storage, doms, order=order)
    c = lbm.Batch(lattice, storage, doms, order=order)
    c.set_schedule(mode="stepwise", xcd_group=1)
    for k in (steps, 2, 1):
        b.step(k)
        c.step(k)
        assert b.t == c.t
        assert torch.equal(b.f64(), c.f64())
    b.close()
    c.close()
