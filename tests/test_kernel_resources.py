"""What the compiler gave the kernels of the built library (CPU): no scratch memory and no spilled vector registers, but for k_direct's
rotated forms of 128 dims; two work-groups of k_attn per CU."""
from __future__ import annotations

import os
import re
import shutil
import struct
import subprocess

import pytest
import yaml

from paper_2502_11517_amd import binding as B

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _kernels(tmp_path):
    """name -> resources, from the notes of the gfx950 code object inside the library"""
    if not os.path.exists(B.library_path()):
        B.build_library()
    lib = open(B.library_path(), "rb").read()
    at = lib.index(b"__CLANG_OFFLOAD_BUNDLE__")
    n, pos = struct.unpack_from("<Q", lib, at + 24)[0], at + 32
    for _ in range(n):  # offset, size, length of the target's name, name
        off, size, length = struct.unpack_from("<QQQ", lib, pos)
        if b"gfx950" in lib[pos + 24:pos + 24 + length]:
            (tmp_path / "code.o").write_bytes(lib[at + off:at + off + size])
        pos += 24 + length
    notes = subprocess.run([READELF, "--notes", str(tmp_path / "code.o")], capture_output=True, text=True, check=True).stdout
    doc = yaml.safe_load(notes[notes.index("---"):notes.index("\n...")])
    return {k[".name"]: k for k in doc["amdhsa.kernels"]}


@pytest.mark.skipif(not os.path.exists(READELF) and not shutil.which(READELF), reason="needs llvm-readelf")
def test_no_kernel_spills_but_the_rotated_ones_of_128_dims(tmp_path):
    kernels = _kernels(tmp_path)
    assert sum("6k_attn" in name for name in kernels) == 28
    for name, k in kernels.items():
        if re.search(r"8k_directI[ft]Li128ELb1E", name):
            assert k[".private_segment_fixed_size"] <= 72
            continue
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name
        if "6k_attn" in name:
            assert k[".vgpr_count"] <= 256 and 2 * k[".group_segment_fixed_size"] <= 160 * 1024, name
        if re.search(r"6k_attnILb[01]ELb[01]ELb0ELb0ELb0ELb0E", name):  # the usual launch
            assert k[".sgpr_spill_count"] <= 4, name
