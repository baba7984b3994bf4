"""Masked grids large enough for compact rows, with masks that have them and masks that do not: against the same
grid of 32 or 96 cells per row, written several times along x, which never has them (test_gpu_compact_rows.py)."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_common import check
from tests.test_gpu_compact_rows import TYPE, _copies, _mask, _sims

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
lbm = pytest.importorskip("paper_2605_27004_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("lattice,storage,shape,times,share,order", [
    ("D3Q19", "f64", (32, 58, 57), 2, 0.3, 3), ("D3Q27", "f64", (32, 35, 34), 4, 0.5, 3),
    ("D3Q27", "f64", (96, 30, 26), 2, 0.95, 2), ("D3Q19", "f64", (32, 27, 25), 10, 0.02, 2),
    ("D3Q19", "f64", (32, 20, 19), 18, 0.5, 3), ("D3Q19", "f32", (96, 50, 47), 2, 0.5, 2),
    ("D3Q27", "f32", (32, 60, 43), 4, 0.05, 3), ("D3Q19", "f64", (32, 90, 60), 4, 0.2, 3),
])
def test_rows_whatever_the_mask(lattice, storage, shape, times, share, order):
    a, b = _sims(lattice, storage, shape, times, share, order)
    for n in (0, 1, 6):
        a.step(n)
        b.step(n)
        assert _copies(a.get_populations().view(TYPE[storage]), b.get_populations().view(TYPE[storage]), shape, times)
    c = _sims(lattice, storage, shape, times, share, order)[1]
    c.set_launch(64, 4)
    c.step(7)
    assert torch.equal(c.get_populations(), b.get_populations())
    snap = b.get_populations()
    b.step(3)
    rho, s, _ = b.moments()
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


def test_compact_rows_match_oracle():
    shape = (64, 58, 57)
    rho, s = W.random_fields(shape, 3, 33)
    wl = W.Workload("D3Q19", shape, W.random_theta(33), "theta", 0.75, 0, rho, s, 0.02)
    wl.meta["mask"] = _mask(shape, 0.4, 33).ravel()
    wl.meta["force"] = np.array([1e-5, -2e-5, 5e-6])
    check(wl, "f64", 12)


@pytest.mark.parametrize("lattice,storage,shape,times,share", [
    ("D3Q19", "f64", (32, 58, 57), 2, 0.3), ("D3Q27", "f64", (32, 20, 19), 18, 0.5), ("D3Q19", "f32", (96, 50, 47), 2, 0.4)])
def test_gradient_whatever_the_mask(lattice, storage, shape, times, share):
    """The sums of a grid written `times` times are that many times the sums of the one."""
    a, b = _sims(lattice, storage, shape, times, share, 3)
    ja, ta, ua, ma = a.grad("kinetic_energy", 8, 4, 5)
    jb, tb, ub, mb = b.grad("kinetic_energy", 8, 4, 5)
    tol = 1e-9 if storage == "f64" else 2e-5
    ta, tb = np.asarray(ta), np.asarray(tb)
    assert abs(jb - times * ja) <= tol * abs(times * ja)
    assert np.abs(tb - times * ta).max() <= tol * np.abs(times * ta).max()
    assert abs(ub - times * ua) <= tol * abs(times * ua)
    nx, ny, nz = shape
    ma, mb = ma.reshape(nz, ny, 1, nx), mb.reshape(nz, ny, times, nx)
    assert (mb - ma).abs().max().item() <= tol * ma.abs().max().item()
