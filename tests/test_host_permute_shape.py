"""Work-groups of exports and imports over long rows: parts that divide the rows where that is faster, else 256 cells.
(No GPU: the launches are listed.)"""
from tests import fake_hip


def test_work_groups_of_long_rows():
    # lattice, storage, extents, masked; work-groups' width of the export, the import and the FP64 export
    cases = [("D2Q9", "bf16", (9792, 1713, 1), False, 64, 256, 64), ("D2Q9", "f32", (2624, 3000, 1), False, 64, 256, 256),
             ("D2Q9", "f64", (640, 4000, 1), False, 128, 256, 256), ("D2Q9", "f32", (2624, 3000, 1), True, 64, 64, 64),
             ("D3Q27", "f16", (384, 64, 64), False, 128, 128, 128), ("D3Q19", "f16", (320, 64, 64), False, 64, 64, 64), ("D3Q19", "f16", (448, 64, 64), False, 64, 256, 64), ("D3Q19", "bf16", (640, 64, 64), False, 128, 256, 128),
             ("D3Q19", "f32", (512, 64, 64), True, 256, 256, 256), ("D3Q19", "f32", (300, 64, 64), False, 256, 256, 256)]
    got = fake_hip.run(f"""
out = []
for lat, st, sh, masked, *_ in {cases!r}:
    c = make(lat, st, sh, masked=masked)
    for call in (lbm.lbm_get_populations, lbm.lbm_set_populations, lbm.lbm_get_f64):
        call(c, 1 << 50)
    out.append([l["grid"] for l in fake.launches()])
    lbm.lbm_destroy(c)
""")
    for (lat, st, (nx, ny, nz), masked, *widths), grids in zip(cases, got):
        assert grids == [-(-nx // w) * -(-ny // (256 // w)) * nz for w in widths], (lat, st, nx, masked)
