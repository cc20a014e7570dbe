"""Registers and scratch memory of the built matrix-core scorer (CPU only: the
kernels' metadata in libspot.so).

Two workgroups of 4 waves share a CU (256 registers a wave, 80 KiB of LDS each); a
kernel that needs more runs one and takes up to 1.7 times as long.  Arrays that
the compiler puts into scratch memory cost more: 3 times, for integer queries and
64-dim heads.
"""
import os
import re
import subprocess

import pytest

from paper_2606_22874_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MARK = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels(tmp_path):
    """{kernel symbol: {metadata field: value}} of every code object in libspot.so."""
    if not os.path.exists(build.SO):
        build.build()
    with open(build.SO, "rb") as f:
        data = f.read()
    out = {}
    for m in re.finditer(re.escape(MARK), data):
        at = data.find(b"\x7fELF", m.start())
        if at < 0:
            continue
        nxt = data.find(MARK, at)
        obj = tmp_path / "code.o"
        obj.write_bytes(data[at:nxt if nxt > 0 else len(data)])
        notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True,
                               text=True).stdout
        for part in re.split(r"\n  - (?=\.)", notes):
            sym = re.search(r"\.symbol: +(\S+)\.kd", part)
            if sym:
                out[sym.group(1)] = {k: int(v) for k, v in
                                     re.findall(r"^ +\.(\w+): +(\d+)$", part, re.M)}
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-readelf")
def test_score_many_registers_and_scratch(tmp_path):
    found = {k: v for k, v in kernels(tmp_path).items() if "score_many_kernel" in k}
    assert len(found) == 40                  # 5 key formats x 2 head sizes x 4 uses
    for name, v in found.items():
        assert v["vgpr_count"] <= 256, (name, v)
        assert v["private_segment_fixed_size"] <= 128, (name, v)   # a few spilled registers
        assert 2 * v["group_segment_fixed_size"] <= 160 * 1024, (name, v)
