"""CPU test of the built library's kernels: no LU elimination kernel and no
kernel that finds inverses from its factors uses scratch memory or spills."""

import os
import re
import subprocess

import pytest

from test_kernel_resources import BIN, LIB


def notes(tmp_path):
    """Kernel name -> (scratch bytes, spilled vector registers)."""
    lib = str(tmp_path / "lib.so")
    os.symlink(LIB, lib)
    subprocess.run([f"{BIN}/llvm-objdump", "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" not in f:
            continue
        txt = subprocess.run([f"{BIN}/llvm-readelf", "--notes", str(tmp_path / f)], check=True, capture_output=True,
                             text=True).stdout
        for k in re.split(r"\n\s*- \.agpr_count", txt)[1:]:
            field = lambda x: re.search(rf"\.{x}:\s*(\S+)", k).group(1)
            out[field("name")] = int(field("private_segment_fixed_size")), int(field("vgpr_spill_count"))
    return out


def test_no_lu_kernel_uses_scratch(tmp_path):
    if not os.path.exists(LIB) or not os.path.exists(f"{BIN}/llvm-objdump"):
        pytest.skip("needs the built library and the ROCm binary tools")
    k = {n: v for n, v in notes(tmp_path).items() if "k_lu_" in n}
    for part in ("k_lu_bandI", "k_lu_band_rowsI", "k_lu_band_rows_long", "k_lu_blocks", "k_lu_rows"):
        assert any(part in n for n in k), part
    assert {n: v for n, v in k.items() if v != (0, 0)} == {}
