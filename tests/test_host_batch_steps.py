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


def test_planning_needs_little_memory():
    """One long, thin domain: cut into runs of a few planes it would be ten million records; the plan counts them
    before it makes any."""
    peak = fake_hip.run("""
b = make_batch("D3Q19", "f32", [(1, 1, 40_000_000)])
lbm.lbm_batch_step(b, 2)
assert all("k_batch_step" in l["name"] for l in fake.launches())
out = int(next(x for x in open("/proc/self/status") if x.startswith("VmHWM")).split()[1]) / 1024
""")
    assert peak < 300, peak  # MiB


def test_schedule_there_and_back():
    out = fake_hip.run("""
out = []
for lat, st, shape in (("D3Q19", "f64", (64, 64, 64)), ("D2Q9", "f32", (40, 30, 1))):
    b = make_batch(lat, st, [shape] * 40)
    names = []
    for kw in ({}, dict(xcd_group=1), dict(), dict(mode="persistent", wg_per_cu=1, chunk_cells=4096), dict()):
        lbm.lbm_batch_set_schedule(b, lbm.make_batch_schedule(**kw))
        fake.launches()
        lbm.lbm_batch_step(b, 6)
        names.append([(l["name"], l["grid"], l["block"]) for l in fake.launches()])
    out.append(names)
""")
    for first, xcd, again, persistent, last in out:
        assert first == again == last and first != xcd
        assert all("k_batch_step" in n for n, _, _ in xcd) and len(xcd) == 6
