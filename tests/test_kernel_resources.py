"""CPU test of the built library's kernels: the LU eliminations use no scratch
memory (the compiler has spilled into one side of a divergent branch of them,
which left the other side's lanes with stale rows)."""

import os
import re
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1709_05660_amd", "libfsimg.so")
BIN = "/opt/rocm/llvm/bin"


def _kernels(tmp_path):
    subprocess.run([f"{BIN}/llvm-objdump", "--offloading", LIB], cwd=tmp_path, check=True, capture_output=True)
    # the extracted images are written beside the input or in the working directory
    out = {}
    for d in (str(tmp_path), os.path.dirname(LIB)):
        for f in sorted(os.listdir(d)):
            if not f.startswith("libfsimg.so."):
                continue
            path = os.path.join(d, f)
            if "gfx950" in f:
                txt = subprocess.run([f"{BIN}/llvm-readelf", "--notes", path], check=True, capture_output=True,
                                     text=True).stdout
                for k in re.split(r"\n\s*- \.agpr_count|\n  - \.", txt)[1:]:
                    name = re.search(r"\.name:\s*(\S+)", k)
                    size = re.search(r"\.private_segment_fixed_size:\s*(\d+)", k)
                    if name and size:
                        out[name.group(1)] = int(size.group(1))
            os.unlink(path)
    return out


def test_lu_kernels_use_no_scratch(tmp_path):
    if not os.path.exists(LIB) or not os.path.exists(f"{BIN}/llvm-objdump"):
        pytest.skip("needs the built library and the ROCm binary tools")
    k = {n: v for n, v in _kernels(tmp_path).items() if re.search(r"k_lu_(blocks|rows|bandI)", n)}
    assert len(k) >= 23
    assert {n: v for n, v in k.items() if v} == {}
