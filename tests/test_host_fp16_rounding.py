"""FP16 steps of a D2Q9 grid round the same way in every kernel that may make them.

On gfx950 the compiler may turn a multiply-add and its conversion to FP16 into one instruction that rounds once
(v_fma_mixlo_f16), where another kernel rounds twice; the results then differ in the last bit now and then.
Steps without walls and steps over gray cells are made by the tile kernels and by the single-step kernels, so in
both all nine conversions have to be of the same kind. This reads the built library's own gfx950 code.
"""
import os
import re
import struct
import subprocess

import pytest

lbm = pytest.importorskip("paper_2605_27004_amd")

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
OBJDUMP = os.path.join(LLVM, "llvm-objdump")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects():
    """The gfx950 code objects in the library, one per source file."""
    data = open(lbm.LIB_PATH, "rb").read()
    for m in re.finditer(MAGIC, data):
        at = m.start()
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        if count > 16:
            continue  # (the text of the magic elsewhere)
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24: p + 24 + n]
            p += 24 + n
            if b"gfx950" in triple:
                yield data[at + off: at + off + size]


def test_fp16_steps_round_alike(tmp_path):
    kinds = {}
    for k, obj in enumerate(_code_objects()):
        path = tmp_path / f"{k}.o"
        path.write_bytes(obj)
        names = subprocess.run([OBJDUMP, "--syms", path], capture_output=True, text=True, check=True).stdout
        # order 2 and 3, plain (0) and gray (2): k_tile<S, order, mode, lanes, cells, row>, k_step<D2Q9, S, order, mode, ..>
        want = re.findall(r"\S*(?:6k_tileIDF16_Li[23]ELi[02]E|6k_stepILi0EDF16_Li[23]ELi[02]E)\S*(?<!\.kd)$", names, re.M)
        if not want:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--disassemble-symbols=" + ",".join(want), path], capture_output=True,
                              text=True, check=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, re.S | re.M):
            once = len(re.findall(r"\bv_fma_mix(?:lo|hi)_f16\b", body))
            twice = len(re.findall(r"\bv_cvt_f16_f32|\bv_cvt_pk_f16|\bv_cvt_pkrtz", body))
            mode = re.search(r"DF16_Li([23])ELi([02])E", name).groups()
            kinds.setdefault(mode, {})[name] = (once, twice)
    assert sorted(kinds) == [("2", "0"), ("2", "2"), ("3", "0"), ("3", "2")]
    for mode, found in kinds.items():
        assert sum("k_tile" in n for n in found) == 3 and sum("k_step" in n for n in found) == 5, found
        for name, (once, twice) in found.items():
            cells = 1 if "k_step" in name or "Li512ELi1E" in name else 2  # cells per lane
            assert (once, twice) in ((9 * cells, 0), (0, 9 * cells)), (name, once, twice)
            # of one kind in all of them
            assert (once == 0) == (next(iter(found.values()))[0] == 0), found
