"""Which D2Q9 grids take several steps per launch: planes do, strips that a tile covers only in small part take
single steps, which every grid has at hand. (No GPU: the launches are listed.)"""
import pytest

from tests import fake_hip

CODE = """
out = []
for st, nx, ny, kw in {grids}:
    c = make("D2Q9", st, (nx, ny, 1), **kw)
    lbm.lbm_step(c, 24)
    out.append(sorted(set("k_tile" if "k_tile" in l["name"] else "k_step" for l in fake.launches())))
    lbm.lbm_destroy(c)
"""
STORAGES = ("f64", "f32", "f16", "bf16")
WALLS = ({}, {"gray": True}, {"force": [1e-5, 0.0]}, {"masked": True})


def _routes(grids):
    return fake_hip.run(CODE.format(grids=grids))


@pytest.mark.parametrize("walls", WALLS, ids=["plain", "gray", "force", "mask"])
def test_strips_take_single_steps(walls):
    shapes = [(4_000_000, 1), (100_000, 1), (400_000, 2), (8, 125_000), (4, 1_000_000), (1, 300_000)]
    grids = [(st, nx, ny, walls) for st in STORAGES for nx, ny in shapes]
    # the longest strip of 16-bit storage: its tiles would be more lanes than one launch may have
    grids.append(("bf16", 238_000_000, 1, walls))
    for g, route in zip(grids, _routes(grids)):
        assert route == ["k_step"], g


@pytest.mark.parametrize("walls", WALLS, ids=["plain", "gray", "force", "mask"])
def test_planes_take_tiles(walls):
    shapes = [(5, 3), (64, 64), (90, 47), (128, 100), (200, 150), (260, 380), (350, 330), (512, 512), (600, 444),
              (1000, 700), (1500, 1103), (3000, 2000), (2896, 2896), (60, 1000), (1000, 60), (700, 30), (30, 700)]
    grids = [(st, nx, ny, walls) for st in STORAGES for nx, ny in shapes
             if not (st == "f16" and ("force" in walls or "masked" in walls))]
    for g, route in zip(grids, _routes(grids)):
        assert route == ["k_tile"], g


def test_two_steps_over_a_middling_plane_are_single_steps():
    out = fake_hip.run("""
out = []
for st, nx, ny in (("f32", 400, 300), ("bf16", 512, 512), ("f32", 512, 512), ("f64", 64, 64), ("f64", 576, 664)):
    c = make("D2Q9", st, (nx, ny, 1))
    row = []
    for n in (2, 3):
        lbm.lbm_step(c, n)
        row.append(["k_tile" in l["name"] for l in fake.launches()])
    out.append(row)
    lbm.lbm_destroy(c)
""")
    single, tiled = [[False, False], [True]], [[True], [True]]
    assert out == [single, single, tiled, tiled, tiled]
