"""Registers of the kernels that are cut for a number of waves per SIMD, from the metadata of the built library: the pull of
the bf16 model at eight waves (64 registers) keeps its row loop in them, or the rows it has in flight wait for scratch."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2303_13775_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> spilled vector registers"""
    if not os.path.exists(os.path.join(LLVM, "llvm-readelf")):
        pytest.skip("needs the ROCm LLVM tools")
    if not os.path.exists(build.LIB):
        build.build()
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(build.LIB, d / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], check=True, capture_output=True, cwd=d)
    spills = {}
    for f in sorted(d.glob("*gfx950")):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(f)], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"\n  - \.", notes):
            name, n = re.search(r"\.name: +(\S+)\n", part), re.search(r"\.vgpr_spill_count: +(\d+)", part)
            if name and n:
                spills[name.group(1)] = int(n.group(1))
    return spills


# rows of a wave: 64 lanes (gradient rows of more than 128 values), 32 and 16
@pytest.mark.parametrize("lanes, allowed", [(64, 0), (32, 1), (16, 1)])
def test_pull_of_bf16_rows_stays_in_its_registers(kernels, lanes, allowed):
    names = [k for k in kernels if f"k_pull_input_gradILi{lanes}ELi4ELb1ELb1E" in k]
    assert len(names) == 1, names
    assert kernels[names[0]] <= allowed
