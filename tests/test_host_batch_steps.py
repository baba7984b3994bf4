"""Batches: calls of one step take the single-step launch, whatever the plan for more. (No GPU: the launches are
listed.)"""
import pytest

from tests import fake_hip


@pytest.mark.parametrize("lattice,storage,shape,kernel", [
    ("D2Q9", "f32", (64, 64, 1), "k_batch_tile"), ("D2Q9", "f64", (16, 20, 1), "k_batch_tile"),
    ("D3Q19", "f64", (64, 64, 64), "k_batch_sweep")])
def test_one_step_is_a_single_step(lattice, storage, shape, kernel):
    out = fake_hip.run(f"""
b = make_batch({lattice!r}, {storage!r}, [{shape!r}] * 40)
out = []
for n in (1, 2, 1, 5):
    lbm.lbm_batch_step(b, n)
    out.append([l["name"] for l in fake.launches()])
""")
    one, two, again, five = out
    assert len(one) == len(again) == 1 and "k_batch_step" in one[0] and one == again
    assert len(two) == 1 and kernel in two[0]
    assert len(five) <= 3 and kernel in five[0]
