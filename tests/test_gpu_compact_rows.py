"""Masked grids whose rows store their fluid cells first (three-dimensional lattices, rows of a multiple
of 64 cells, FP64 or large FP32 grids) against grids that do not.

A periodic grid of 32 or 96 cells per row keeps every cell in its place; the same grid written twice
or more along x has rows of 64 to 576 cells and stores the fluid cells first. Both hold the same values,
bit for bit.
"""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lbm = pytest.importorskip("paper_2605_27004_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _mask(shape, share, seed):
    """Random solid cells, with a whole solid row, a whole fluid row, rows of one fluid cell at either
    end, and rows with one solid cell at either end."""
    nx, ny, nz = shape
    m = (np.random.default_rng(seed).uniform(size=(nz, ny, nx)) < share).astype(np.uint8)
    m[0, 0] = 1
    m[0, 1] = 0
    m[1, 0] = 1
    m[1, 0, 0] = 0
    m[1, 1] = 1
    m[1, 1, -1] = 0
    m[2, 0] = 0
    m[2, 0, 0] = 1
    m[2, 1] = 0
    m[2, 1, -1] = 1
    return m


def _sims(lattice, storage, shape, times, share, order, seed=31):
    """The grid and its `times`-fold copy along x."""
    nx, ny, nz = shape
    rho, s = W.random_fields(shape, 3, seed)
    rho, s = rho.reshape(nz, ny, nx), s.reshape(3, nz, ny, nx)
    m = _mask(shape, share, seed)
    out = []
    for t in (1, times):
        p = lbm.make_params(lattice, storage, (t * nx, ny, nz), W.random_theta(seed), "theta", 0.8, order,
                            force=[1e-4, -3e-5, 5e-5], masked=True)
        out.append(lbm.Simulation(p, np.ascontiguousarray(np.tile(rho, (1, 1, t)).ravel()),
                                  np.ascontiguousarray(np.tile(s, (1, 1, 1, t)).reshape(3, -1)),
                                  mask=np.ascontiguousarray(np.tile(m, (1, 1, t)).ravel())))
    return out


TYPE = {"f64": torch.float64, "f32": torch.float32}


def _copies(a, b, shape, times):
    """Every copy in b, a field of the wide grid, is a."""
    nx, ny, nz = shape
    a, b = a.reshape(-1, nz, ny, 1, nx), b.reshape(-1, nz, ny, times, nx)
    assert bool(torch.isfinite(a.double()).all())
    return all(torch.equal(a[:, :, :, 0], b[:, :, :, t]) for t in range(times))


@pytest.mark.parametrize("lattice,storage,shape,times,share,order", [
    ("D3Q19", "f64", (32, 5, 4), 2, 0.3, 3), ("D3Q27", "f64", (32, 3, 3), 4, 0.5, 3),
    ("D3Q27", "f64", (96, 6, 5), 2, 0.95, 2), ("D3Q19", "f64", (32, 4, 7), 10, 0.02, 2),
    ("D3Q19", "f64", (32, 2, 3), 18, 0.5, 3), ("D3Q27", "f32", (32, 60, 43), 4, 0.4, 3),
    ("D3Q19", "f32", (96, 50, 47), 2, 0.1, 2), ("D3Q19", "f32", (32, 40, 21), 18, 0.6, 3),
])
def test_rows_of_fluid_cells(lattice, storage, shape, times, share, order):
    a, b = _sims(lattice, storage, shape, times, share, order)
    for n in (0, 1, 6):
        a.step(n)
        b.step(n)
        assert _copies(a.get_populations().view(TYPE[storage]), b.get_populations().view(TYPE[storage]), shape, times)
    for shaped in ((64, 1), (192, 1), (64, 4)):
        c = _sims(lattice, storage, shape, times, share, order)[1]
        c.set_launch(*shaped)
        c.step(7)
        assert torch.equal(c.get_populations(), b.get_populations())
    # export and import: continuing from a restored state reproduces the run
    snap = b.get_populations()
    b.step(3)
    rho, s, _ = b.moments()
    rho, s = rho.clone(), s.clone()
    b.set_populations(snap)
    assert torch.equal(b.get_populations(), snap)
    b.step(3)
    rho2, s2, tot = b.moments()
    assert torch.equal(rho, rho2) and torch.equal(s, s2)
    a.step(3)
    rho1, s1, tot1 = a.moments()
    assert _copies(rho1, rho2, shape, times) and _copies(s1, s2, shape, times)
    want = np.array(tot1) * times
    assert np.abs(np.array(tot) - want).max() <= 1e-12 * np.abs(want).max()


def test_rows_of_fluid_cells_of_more_than_4_gib():
    shape, times, storage = (32, 560, 560), 2, "f64"
    a, b = _sims("D3Q27", storage, shape, times, 0.3, 3)
    a.step(2)
    b.step(2)
    assert _copies(a.get_populations().view(TYPE[storage]), b.get_populations().view(TYPE[storage]), shape, times)


@pytest.mark.parametrize("lattice,storage,shape", [("D3Q19", "f64", (64, 7, 5)), ("D3Q27", "f64", (192, 5, 4))])
def test_rows_of_fluid_cells_match_oracle(lattice, storage, shape):
    rho, s = W.random_fields(shape, 3, 33)
    wl = W.Workload(lattice, shape, W.random_theta(33), "theta", 0.75, 0, rho, s, 0.02)
    wl.meta["mask"] = _mask(shape, 0.3, 33).ravel()
    wl.meta["force"] = np.array([1e-5, -2e-5, 5e-6])
    check(wl, storage, 30)


@pytest.mark.parametrize("lattice,storage,shape,times,objective", [
    ("D3Q19", "f64", (32, 5, 4), 2, "kinetic_energy"), ("D3Q27", "f64", (32, 4, 4), 6, "kinetic_energy"),
    ("D3Q19", "f32", (96, 50, 47), 2, "kinetic_energy"), ("D3Q27", "f64", (32, 3, 4), 10, "flux"),
])
def test_gradient_over_rows_of_fluid_cells(lattice, storage, shape, times, objective):
    """The sums of a grid written `times` times are that many times the sums of the one (the flux through
    one plane has the same value, its derivatives too: every plane of the copy is one of the grid, and
    a cell's share is spread over them)."""
    a, b = _sims(lattice, storage, shape, times, 0.3, 3)
    k = times if objective == "kinetic_energy" else 1
    ja, ta, ua, ma = a.grad(objective, 12, 4, 5)
    jb, tb, ub, mb = b.grad(objective, 12, 4, 5)
    tol = 1e-9 if storage == "f64" else 2e-5
    ta, tb = np.asarray(ta), np.asarray(tb)
    assert abs(jb - k * ja) <= tol * abs(k * ja)
    assert np.abs(tb - k * ta).max() <= tol * np.abs(k * ta).max()
    assert abs(ub - k * ua) <= tol * abs(k * ua)
    # a cell's own sensitivity: of the energy the same in every copy, of the flux shared out over them
    nx, ny, nz = shape
    ma, mb = ma.reshape(nz, ny, 1, nx), mb.reshape(nz, ny, times, nx)
    got = mb if k == times else mb.sum(dim=2, keepdim=True)
    assert (got - ma).abs().max().item() <= tol * ma.abs().max().item()
