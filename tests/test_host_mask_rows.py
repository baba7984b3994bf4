"""Which masked grids store their rows compact: the mask decides, by its solid cells and their runs along x. (No GPU:
the launches are listed; the counts are made up.)"""
from tests import fake_hip

CODE = """
out = []
for lat, st, (nx, ny, nz), solid, runs, rec in {grids!r}:
    n = nx * ny * nz
    fake.launches()
    fake.result(solid * n, runs * n)
    fake.capture(rec)
    p = lbm.make_params(lat, st, (nx, ny, nz), None, "theta", 0.8, 3, masked=True)
    c = lbm.lbm_init(p, A, B, SCRATCH, RHO, S, MASK, None)
    fake.result()
    fake.capture(False)
    names = [l["name"] for l in fake.launches()]
    lbm.lbm_step(c, 1)
    step = fake.launches()[0]["name"]
    out.append([any("k_row_index" in x for x in names), any("k_links" in x for x in names),
                any("k_mask_stats" in x for x in names), step])
    lbm.lbm_destroy(c)
"""


def test_the_mask_decides():
    small, large, wide = (64, 64, 64), (128, 128, 128), (320, 128, 128)
    # lattice, storage, extents, solid cells and runs per cell, recorded; compact rows, mask counted
    cases = [("D3Q19", "f32", large, 0.0, 0.0, False, False, True), ("D3Q19", "f32", large, 0.40, 0.023, False, True, True),
             ("D3Q19", "f32", large, 0.10, 0.09, False, False, True), ("D3Q19", "f32", large, 0.22, 0.17, False, False, True),
             ("D3Q27", "f32", wide, 0.30, 0.21, False, True, True), ("D3Q27", "f32", large, 0.22, 0.0, False, True, True),
             ("D3Q19", "f64", large, 0.016, 0.0, False, False, True), ("D3Q19", "f64", large, 0.12, 0.01, False, True, True),
             ("D3Q19", "f64", large, 0.05, 0.047, False, False, True), ("D3Q27", "f64", small, 0.17, 0.14, False, False, True),
             ("D3Q27", "f64", small, 0.30, 0.21, False, True, True), ("D3Q19", "f64", (128, 28, 28), 0.40, 0.02, False, True, True),
             ("D3Q19", "f64", (128, 28, 28), 0.22, 0.01, False, False, True), ("D3Q19", "f64", (64, 24, 24), 0.6, 0.03, False, False, False),
             ("D3Q19", "f32", small, 0.6, 0.03, False, False, False), ("D3Q27", "f16", large, 0.6, 0.03, False, False, False),
             # a stream that is being recorded cannot be waited for
             ("D3Q19", "f32", large, 0.40, 0.023, True, False, False)]
    got = fake_hip.run(CODE.format(grids=[c[:6] for c in cases]))
    for c, (rows, links, counted, step) in zip(cases, got):
        assert (rows, links, counted) == (c[6], not c[6], c[7]), c
        pull = step.split("k_step<")[1].split(">")[0].split(",")[4] if "k_step<" in step else ""
        if pull:
            assert (int(pull) == 3) == c[6], (c, step)  # kPullCompact
