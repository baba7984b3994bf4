"""Step launches of runs of consecutive cells (rows that are no multiple of 64 cells) and with cached
stores: bit for bit the boxes with non-temporal stores that a launch shaped by the caller takes.

Shapes: rows shorter and longer than a work-group, of one cell, of whole cache lines and not, z-planes
that are no multiple of 256 cells, and both sides of the size at which stores stay in the caches.
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


@pytest.mark.parametrize("lattice,storage,shape,walls,order", [
    ("D3Q19", "f16", (33, 31, 9), "none", 3), ("D3Q27", "f16", (129, 50, 10), "mask", 3),
    ("D3Q27", "bf16", (300, 7, 12), "none", 2), ("D3Q19", "f32", (1, 9, 40), "gray", 3),
    ("D3Q19", "f32", (65, 17, 20), "gray", 2), ("D3Q27", "f32", (77, 40, 15), "mask", 3),
    ("D3Q27", "f64", (50, 21, 14), "gray", 3), ("D3Q19", "f64", (17, 16, 16), "mask", 2),
    ("D3Q19", "f32", (96, 40, 40), "gray", 3), ("D3Q19", "f16", (128, 96, 96), "gray", 3),
    ("D3Q27", "f16", (320, 12, 10), "none", 3), ("D3Q19", "f32", (160, 180, 110), "gray", 3),
    ("D3Q19", "f32", (57, 47, 40), "gray", 3), ("D3Q19", "f16", (62, 80, 80), "gray", 2),
])
def test_launch_of_runs_is_launch_of_boxes(lattice, storage, shape, walls, order):
    rho, s = W.random_fields(shape, 3, 17)
    rng = np.random.default_rng(17)
    n = int(np.prod(shape))
    mask = None
    if walls == "mask":
        mask = (rng.uniform(size=n) < 0.3).astype(np.uint8)
    elif walls == "gray":
        mask = rng.uniform(0.0, 0.4, n).astype(np.float32)
    p = lbm.make_params(lattice, storage, shape, W.random_theta(17), "theta", 0.8, order,
                        force=None if walls == "none" else [1e-4, 0.0, -5e-5], masked=walls == "mask",
                        gray=walls == "gray")
    out = []
    for shaped in (False, True):
        sim = lbm.Simulation(p, rho, s, mask=mask)
        if shaped:
            sim.set_launch(64, 4)
        sim.step(9)
        out.append(sim.get_populations().cpu().numpy())
        sim.close()
    assert np.array_equal(*out)
