"""The two-step pass of periodic three-dimensional grids: bit for bit two single steps, and the oracle.

The library takes steps two at a time on grids of about 100^3 cells and more (an odd number ends
with a single step); a launch shape set by the caller keeps every step a single one. The grids here
are the smallest of their kind on which the rule picks the two-step pass: rows shorter than a
tile, ragged tiles in x and y, uneven z segments, and whole tiles.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lbm = pytest.importorskip("paper_2605_27004_amd")

from tests.gpu_common import check, gpu_run  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("lattice,storage,shape,order,steps", [
    ("D3Q19", "f32", (64, 299, 31), 3, 5),    # rows of one tile, uneven segments
    ("D3Q19", "f32", (192, 96, 64), 2, 6),    # whole cache lines, order 2
    ("D3Q19", "f64", (45, 90, 250), 3, 5),    # rows shorter than a tile, 64-wide tiles ragged in y
    ("D3Q19", "f64", (96, 100, 97), 3, 4),    # 32-wide tiles
    ("D3Q27", "f32", (200, 190, 99), 3, 5),   # ragged in x and y, two segments
    ("D3Q27", "f64", (130, 111, 83), 3, 5),
])
def test_two_step_pass_is_two_steps(lattice, storage, shape, order, steps):
    d = W.DIMS[lattice]
    rho, s = W.random_fields(shape, d, 13)
    wl = W.Workload(lattice, shape, W.random_theta(13), "theta", 0.75, 0, rho, s, 0.02, order=order)
    g, _, _ = check(wl, storage, steps)
    single = gpu_run(wl, storage, steps, block=(64, 4, 0))
    assert np.array_equal(g["f"], single["f"])
    assert g["totals"] == single["totals"]
