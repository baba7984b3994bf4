"""Steps of long, thin D2Q9 grids, on both sides of the line between tiles and single steps: bit for bit the single
steps of a launch that the caller has shaped."""
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


@pytest.mark.parametrize("storage,shape,walls", [
    ("f32", (70001, 1), "none"), ("f64", (1, 9001), "gray"), ("f16", (8, 12500), "none"), ("bf16", (20011, 4), "force"),
    ("f32", (20011, 30), "mask"), ("f64", (24, 30011), "none"), ("bf16", (64, 6001), "gray"), ("f32", (8192, 1), "none")])
def test_strip_steps_are_single_steps(storage, shape, walls):
    shape = shape + (1,)
    rho, s = W.random_fields(shape, 2, 11)
    rng = np.random.default_rng(11)
    n = int(np.prod(shape))
    mask = None
    if walls == "mask":
        mask = (rng.uniform(size=n) < 0.3).astype(np.uint8)
    elif walls == "gray":
        mask = rng.uniform(0.0, 0.4, n).astype(np.float32)
    p = lbm.make_params("D2Q9", storage, shape, W.config1_theta(), "theta", 0.8,
                        force=None if walls == "none" else [1e-4, -5e-5], masked=walls == "mask", gray=walls == "gray")
    sims = [lbm.Simulation(p, rho, s, mask=mask) for _ in range(2)]
    sims[1].set_launch(64, 4)
    for k in (1, 13):
        for sim in sims:
            sim.step(k)
        assert torch.equal(*(sim.get_populations() for sim in sims))
    for sim in sims:
        sim.close()
