"""Steps recorded into a graph: as many launches as leave the state in the buffer that one launch per step
would, so that a graph of an even number of steps can be replayed. (No GPU: the launches are listed.)"""
import pytest

from tests import fake_hip

CONTEXTS = {
    "sweep": "make('D3Q19', 'f32', (128, 128, 128))",
    "tile": "make('D2Q9', 'f64', (64, 64, 1))",
    "single": "make('D3Q19', 'f16', (32, 32, 32))",
    "batch-sweep": "make_batch('D3Q19', 'f64', [(64, 64, 64)] * 40)",
    "batch-tile": "make_batch('D2Q9', 'f32', [(64, 64, 1)] * 40)",
    "batch-single": "make_batch('D3Q19', 'f16', [(16, 16, 16)] * 3)",
}


@pytest.mark.parametrize("kind", CONTEXTS)
def test_recorded_launches_keep_the_parity(kind):
    out = fake_hip.run(f"""
c = {CONTEXTS[kind]}
step = lbm.lbm_batch_step if {kind.startswith("batch")} else lbm.lbm_step
out = []
for n in list(range(41)) + [97, 98, 1000]:
    for on in (False, True):
        fake.capture(on)
        step(c, n)
        out.append([n, on, [l["args"][:2] for l in fake.launches()]])
    fake.capture(False)
""")
    cur, other = 1 << 40, 2 << 40
    plain = {n: len(launches) for n, on, launches in out if not on}
    for n, on, launches in out:
        for src, dst in launches:  # each launch goes on from the last one's state
            assert (src, dst) == (cur, other)
            cur, other = other, cur
        if on:
            assert (len(launches) - n) % 2 == 0
            assert plain[n] <= len(launches) <= plain[n] + 1
    if kind not in ("single", "batch-single"):
        assert plain[40] <= 20
