"""Runs host code of the library without a GPU, against a stand-in for the HIP runtime (fake_hip.cpp): which
kernels a call launches, with which arguments, and what happens when a launch fails (not a test module).

    run(code)    runs ``code`` in a process of its own, with `lbm` (the package), `fake` (below) and `make`
                 / `make_batch` (contexts on made-up device addresses) at hand, and returns the JSON value
                 that it leaves in `out`.
"""
import functools
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@functools.lru_cache(maxsize=1)
def _dir():
    return tempfile.TemporaryDirectory()


@functools.lru_cache(maxsize=1)
def _build():
    path = os.path.join(_dir().name, "libamdhip64.so.7")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    "-Wl,-soname,libamdhip64.so.7", os.path.join(HERE, "fake_hip.cpp"), "-o", path], check=True)
    return path


PRELUDE = """
import ctypes, json, sys, types
fake_lib = ctypes.CDLL({path!r}, ctypes.RTLD_GLOBAL)
sys.modules["torch"] = types.ModuleType("torch")   # the binding imports it for its HIP runtime only
sys.path.insert(0, {root!r})
import paper_2605_27004_amd as lbm
fake_lib.fake_name.restype = ctypes.c_char_p
for f in ("fake_grid", "fake_block", "fake_arg"):
    getattr(fake_lib, f).restype = ctypes.c_uint64

class fake:
    capture = staticmethod(lambda on: fake_lib.fake_capture(int(on)))
    fail = staticmethod(lambda name, after=0: fake_lib.fake_fail(name.encode(), after))
    @staticmethod
    def result(*values):  # of the next sums over work-groups
        fake_lib.fake_result((ctypes.c_double * len(values))(*values), len(values))
    @staticmethod
    def launches(clear=True):
        out = []
        for i in range(fake_lib.fake_count()):
            out.append(dict(name=fake_lib.fake_name(i).decode(), grid=fake_lib.fake_grid(i),
                            block=fake_lib.fake_block(i), args=[fake_lib.fake_arg(i, a) for a in range(8)]))
        if clear:
            fake_lib.fake_clear()
        return out

A, B, SCRATCH, RHO, S, MASK = (k << 40 for k in range(1, 7))

def make(lattice, storage, shape, order=3, masked=False, gray=False, force=None):
    p = lbm.make_params(lattice, storage, shape, None, "theta", 0.8, order, force=force, masked=masked, gray=gray)
    c = lbm.lbm_init(p, A, B, SCRATCH, RHO, S, MASK if masked or gray else None, None)
    fake_lib.fake_clear()
    return c

def make_batch(lattice, storage, shapes, order=3):
    theta = [[1 / 3, 0, 0], [0, 1 / 3, 0], [0, 0, 1 / 3]]
    doms = [dict(shape=tuple(s), tensor=theta, tensor_kind="theta", tau=0.8) for s in shapes]
    b = lbm.lbm_batch_init(lbm.make_batch_params(lattice, storage, doms, order), A, B, SCRATCH, RHO, S, None)
    fake_lib.fake_clear()
    return b

out = None
"""


def run(code, timeout=120):
    text = PRELUDE.format(path=_build(), root=ROOT) + code + "\nprint('RESULT ' + json.dumps(out), flush=True)\n"
    r = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=timeout)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    line = [x for x in r.stdout.splitlines() if x.startswith("RESULT ")][-1]
    return json.loads(line[len("RESULT "):])
