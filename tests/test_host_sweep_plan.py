"""Which three-dimensional grids take two steps in a pass: not those whose low tiles would take longer than two
single steps. (No GPU: the launches are listed.)"""
from tests import fake_hip


def test_small_grids_take_the_faster_way():
    single = [("D3Q19", "f64", (64, 48, 54)), ("D3Q19", "f64", (64, 42, 45)), ("D3Q19", "f64", (64, 64, 52)),
              ("D3Q19", "f64", (64, 48, 75)), ("D3Q19", "f32", (48, 48, 48)), ("D3Q27", "f64", (64, 64, 64)),
              ("D3Q27", "f64", (64, 99, 60)), ("D3Q19", "f32", (100, 100, 100)), ("D3Q27", "f32", (150, 101, 75))]
    two = [("D3Q19", "f64", (64, 64, 64)), ("D3Q19", "f32", (64, 64, 64)), ("D3Q19", "f64", (64, 104, 58)), ("D3Q19", "f32", (64, 69, 83)),
           ("D3Q19", "f32", (128, 128, 128)), ("D3Q19", "f64", (250, 190, 130)), ("D3Q27", "f64", (64, 108, 81)),
           ("D3Q27", "f32", (128, 158, 131)), ("D3Q19", "f32", (256, 256, 256))]
    routes = fake_hip.run(f"""
out = []
for lat, st, sh in {single + two!r}:
    c = make(lat, st, tuple(sh))
    lbm.lbm_step(c, 2)
    out.append([l["name"] for l in fake.launches()])
    lbm.lbm_destroy(c)
""")
    for g, names in zip(single + two, routes):
        assert ("k_sweep" in names[0]) == (g in two), (g, names)
        assert len(names) == (1 if g in two else 2)
