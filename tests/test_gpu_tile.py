"""Several steps of a D2Q9 grid in one launch: bit for bit the single steps, and the oracle.

A launch shape set by the caller keeps every step a launch of its own, which is the reference here.
The grids take each of the tile shapes, leave ragged tiles in x and y, and are smaller than a tile
and its rim (the rim then wraps around the grid more than once).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lbm = pytest.importorskip("paper_2605_27004_amd")

from tests.gpu_common import check  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(storage, shape, order, walls, steps, single):
    rho, s = W.random_fields(shape, 2, 7)
    rng = np.random.default_rng(7)
    n = int(np.prod(shape))
    mask = None
    if walls == "mask":
        mask = (rng.uniform(size=n) < 0.3).astype(np.uint8)
    elif walls == "gray":
        mask = rng.uniform(0.0, 0.4, n).astype(np.float32)
    p = lbm.make_params("D2Q9", storage, shape, W.config1_theta(), "theta", 0.8, order,
                        force=None if walls == "none" else [1e-4, -5e-5], masked=walls == "mask",
                        gray=walls == "gray")
    sim = lbm.Simulation(p, rho, s, mask=mask)
    if single:
        sim.set_launch(64, 4)
    out = []
    for k in steps:
        sim.step(k)
        out.append(sim.get_populations().cpu().numpy())
    assert sim.t == sum(steps)
    sim.close()
    return out


@pytest.mark.parametrize("storage,shape,order,walls", [
    ("f64", (64, 64, 1), 3, "none"), ("f32", (5, 3, 1), 3, "force"), ("f16", (61, 47, 1), 2, "gray"),
    ("f32", (61, 47, 1), 3, "mask"), ("bf16", (300, 521, 1), 3, "none"), ("f64", (515, 300, 1), 3, "mask"),
    ("f32", (512, 512, 1), 3, "gray"), ("f32", (1500, 1103, 1), 3, "none"), ("f16", (1111, 1500, 1), 3, "none"),
    ("f64", (1200, 700, 1), 2, "gray"), ("bf16", (90, 1300, 1), 3, "mask"),
])
def test_tiled_steps_are_single_steps(storage, shape, order, walls):
    for a, b in zip(_run(storage, shape, order, walls, (1, 2, 5, 17), False),
                    _run(storage, shape, order, walls, (1, 2, 5, 17), True)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("storage,shape", [("f64", (330, 270, 1)), ("f32", (1030, 900, 1))])
def test_tiled_steps_match_oracle(storage, shape):
    rho, s = W.random_fields(shape, 2, 9)
    check(W.Workload("D2Q9", shape, W.config1_theta(), "theta", 0.75, 0, rho, s, 0.02), storage, 23)
