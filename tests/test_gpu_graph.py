"""A recorded call of an even number of steps, replayed with other work in between, goes on from the state that the
last replay left, as the same calls made one by one do."""
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


def _replayed(make, state, n):
    side = torch.cuda.Stream()
    eager, rec = make(side), make(side)
    graph = torch.cuda.CUDAGraph()
    for k in (eager, rec):
        k.step(3)
    side.synchronize()
    with torch.cuda.graph(graph, stream=side):
        rec.step(n)
    for _ in range(3):
        with torch.cuda.stream(side):
            graph.replay()
            eager.step(n)
            a, b = state(rec), state(eager)
        side.synchronize()
        assert torch.equal(a, b)
        with torch.cuda.stream(side):
            for k in (eager, rec):
                k.step(1)
                k.step(1)
        side.synchronize()


@pytest.mark.parametrize("lattice,storage,shape,n", [
    ("D3Q19", "f32", (192, 96, 64), 2), ("D3Q27", "f64", (130, 111, 83), 6), ("D2Q9", "f64", (64, 64, 1), 8),
    ("D2Q9", "f32", (600, 700, 1), 4), ("D3Q19", "f16", (64, 32, 20), 4)])
def test_recorded_steps(lattice, storage, shape, n):
    d = W.DIMS[lattice]
    rho, s = W.random_fields(shape, d, 3)
    p = lbm.make_params(lattice, storage, shape, W.config1_theta() if d == 2 else W.random_theta(3), "theta", 0.8)
    _replayed(lambda st: lbm.Simulation(p, rho, s, stream=st), lambda k: k.get_populations(), n)


@pytest.mark.parametrize("lattice,edges,n", [("D3Q19", (40, 64), 2), ("D2Q9", (16, 64), 6)])
def test_recorded_batch_steps(lattice, edges, n):
    d = W.DIMS[lattice]
    rng = np.random.default_rng(5)
    doms = []
    for i in range(40):
        sh = tuple(int(v) for v in rng.integers(*edges, d)) + ((1,) if d == 2 else ())
        rho, s = W.random_fields(sh, d, i)
        doms.append(dict(shape=sh, tensor=W.config1_theta() if d == 2 else W.random_theta(i), tensor_kind="theta",
                         tau=0.8, rho=rho, s=s))
    _replayed(lambda st: lbm.Batch(lattice, "f64", doms, stream=st), lambda k: k.f64(), n)
