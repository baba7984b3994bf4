"""Several steps of every plane of a batch in one launch, with work-groups of 512 and of 1,024 lanes: bit for bit the
single steps of the XCD-placed order, which are never taken together."""
import numpy as np
import pytest

import workloads as W
from tests.batch_planes import CASES, planes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lbm = pytest.importorskip("paper_2605_27004_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("storage,count,lo,hi,order,lanes,steps", CASES)
def test_launch_of_several_steps_is_single_steps(storage, count, lo, hi, order, lanes, steps):
    rng = np.random.default_rng(43)
    doms = []
    for i, shape in enumerate(planes(count, lo, hi)):
        rho, s = W.random_fields(shape, 2, 300 + i)
        doms.append(dict(shape=shape, tensor=W.config1_theta(), tensor_kind="theta", tau=float(rng.uniform(0.6, 1.4)),
                         rho=rho, s=s))
    b = lbm.Batch("D2Q9", storage, doms, order=order)
    c = lbm.Batch("D2Q9", storage, doms, order=order)
    c.set_schedule(mode="stepwise", xcd_group=1)
    for k in (steps, 1, steps + 1, 2 * steps - 1, 2):
        b.step(k)
        c.step(k)
        assert torch.equal(b.f64(), c.f64())
    b.close()
    c.close()


def test_totals_of_many_domains():
    """Totals of more domains than a pinned place holds, and of fewer: the same numbers from the same domains."""
    rho, s = W.random_fields((5, 4, 1), 2, 7)
    dom = dict(shape=(5, 4, 1), tensor=W.config1_theta(), tensor_kind="theta", tau=0.8, rho=rho, s=s)
    few, many = lbm.Batch("D2Q9", "f64", [dom] * 3), lbm.Batch("D2Q9", "f64", [dom] * 1100)
    for b in (few, many):
        b.step(5)
    a, c = few.moments()[2], many.moments()[2]
    assert all(row == a[0] for row in a) and len(c) == 1100 and all(row == a[0] for row in c)
    few.close()
    many.close()
