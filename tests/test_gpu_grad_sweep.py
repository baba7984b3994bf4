"""Gradients over a periodic grid that takes two steps in a pass: its forward steps, checkpoints and recomputed segments
give bit for bit what single steps do."""
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


@pytest.mark.parametrize("lattice,storage,shape", [
    ("D3Q19", "f32", (192, 96, 64)), ("D3Q19", "f64", (96, 100, 97)), ("D3Q27", "f64", (130, 111, 83))])
@pytest.mark.parametrize("nsteps,every", [(9, 4), (7, 3), (6, 2), (5, 20)])
def test_gradient_over_two_step_passes(lattice, storage, shape, nsteps, every):
    rho, s = W.random_fields(shape, 3, 23)
    p = lbm.make_params(lattice, storage, shape, W.random_theta(23), "theta", 0.8)
    sims = [lbm.Simulation(p, rho, s) for _ in range(2)]
    sims[1].set_launch(64, 4)  # single steps
    for sim in sims:
        sim.step(2)
    (ja, ta, ua, ma), (jb, tb, ub, mb) = (sim.grad("kinetic_energy", nsteps, every) for sim in sims)
    assert ja == jb and ua == ub and np.array_equal(ta, tb) and torch.equal(ma, mb)
    assert torch.equal(*(sim.get_populations() for sim in sims)) and sims[0].t == nsteps + 2
    for sim in sims:
        sim.close()
