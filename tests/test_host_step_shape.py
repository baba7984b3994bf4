"""How a step over rows that are no multiple of 64 cells is launched: runs of 256 consecutive cells on every lattice,
storage and wall model, with non-temporal stores where the two arrays come near the L2s' size. (No GPU: the
launches are listed.)"""
import re

from tests import fake_hip

RUNS, CACHED, NONTEMPORAL = 2, 0, 2  # PullKind, cache policies


def test_runs_and_their_stores():
    grids = [("D3Q19", "f16", (57, 47, 77), "gray", NONTEMPORAL), ("D3Q19", "bf16", (60, 50, 70), "force", NONTEMPORAL),
             ("D3Q27", "f16", (36, 61, 60), "masked", NONTEMPORAL), ("D3Q19", "f32", (50, 50, 50), "gray", NONTEMPORAL),
             ("D3Q19", "f16", (62, 80, 80), "gray", CACHED), ("D3Q19", "f32", (57, 47, 77), "gray", CACHED),
             ("D3Q19", "f32", (60, 30, 30), "gray", CACHED), ("D3Q27", "f32", (129, 100, 90), "masked", CACHED),
             ("D3Q19", "f64", (200, 150, 100), "gray", NONTEMPORAL), ("D3Q19", "f32", (250, 190, 130), "gray", CACHED),
             ("D3Q19", "f64", (250, 190, 130), "gray", CACHED), ("D3Q19", "f32", (96, 200, 200), "gray", NONTEMPORAL)]
    names = fake_hip.run(f"""
out = []
for lat, st, sh, walls, _ in {grids!r}:
    kw = dict(force=[1e-5, 0.0, 0.0]) if walls == "force" else {{walls: True}}
    c = make(lat, st, sh, **kw)
    lbm.lbm_step(c, 1)
    out.append(fake.launches()[0]["name"])
    lbm.lbm_destroy(c)
""")
    for g, name in zip(grids, names):
        # k_step<lattice, storage, order, mode, pull, store policy>, demangled or (16-bit storage) mangled
        args = re.search(r"k_step<(.*?)>", name)
        if args:
            pull, store = (int(v) for v in args.group(1).split(",")[-2:])
        else:
            pull, store = (int(v) for v in re.findall(r"Li(\d+)E", name.split("k_step", 1)[1].split("Ev", 1)[0])[-2:])
        assert (pull, store) == (RUNS, g[4]), (g, name)
