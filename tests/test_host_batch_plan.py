"""Lanes and steps that the launch of several steps takes for the batches of planes in batch_planes.py. (No GPU: the
launches are listed.)"""
import pytest

from tests import fake_hip
from tests.batch_planes import CASES, planes


@pytest.mark.parametrize("storage,count,lo,hi,order,lanes,steps", CASES)
def test_plan_of_planes(storage, count, lo, hi, order, lanes, steps):
    got = fake_hip.run(f"""
b = make_batch("D2Q9", {storage!r}, {planes(count, lo, hi)!r}, {order})
lbm.lbm_batch_step(b, {3 * steps})
out = [[l["name"], l["block"], l["args"][5]] for l in fake.launches()]
""")
    assert len(got) == 3
    for name, block, k in got:
        assert "k_batch_tile" in name and block == lanes and k == steps
