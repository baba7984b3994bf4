"""Every kernel that the plan for several steps of a D2Q9 grid can pick -- storage, order, wall model, tile -- bit for
bit the single steps, both the default launch's and those of a launch that the caller has shaped."""
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


# up to 8,192, 100,000 and 400,000 cells, and more: the sizes at which the plan changes its tile
@pytest.mark.parametrize("shape", [(61, 47), (211, 190), (520, 411), (677, 631)])
@pytest.mark.parametrize("walls", ["none", "gray", "mask", "force"])
@pytest.mark.parametrize("order", [2, 3])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
def test_tiles_are_single_steps(storage, order, walls, shape):
    shape = shape + (1,)
    rho, s = W.random_fields(shape, 2, 19)
    rng = np.random.default_rng(19)
    n = int(np.prod(shape))
    mask = None
    if walls == "mask":
        mask = (rng.uniform(size=n) < 0.25).astype(np.uint8)
    elif walls == "gray":
        mask = rng.uniform(0.0, 0.5, n).astype(np.float32)
    p = lbm.make_params("D2Q9", storage, shape, W.config1_theta(), "theta", 0.7, order,
                        force=None if walls == "none" else [2e-4, -1e-4], masked=walls == "mask", gray=walls == "gray")
    many, ones, boxes = (lbm.Simulation(p, rho, s, mask=mask) for _ in range(3))
    boxes.set_launch(64, 4)
    for k in (13, 8):
        many.step(k)
        boxes.step(k)
        for _ in range(k):
            ones.step(1)
        want = ones.get_populations()
        assert torch.equal(many.get_populations(), want)
        assert torch.equal(boxes.get_populations(), want)
    for sim in (many, ones, boxes):
        sim.close()
