"""Registers of the built bunch kernels (CPU: the code object's own notes).

The plain bunch kernels hold their state in the 128 vector registers that 16 waves leave
a lane: no scratch, no spilled vector register."""
import os
import shutil
import subprocess

import pytest

from paper_2006_14927_amd import ckv

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def notes(tmp_path_factory):
    if not os.path.exists(ckv.LIB_PATH) or not os.path.exists(f"{LLVM}/llvm-objdump"):
        pytest.skip("needs the built library and llvm-objdump")
    d = tmp_path_factory.mktemp("co")
    shutil.copy(ckv.LIB_PATH, d / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    kernels, cur = {}, {}
    for f in sorted(d.glob("lib.so.*gfx950")):
        text = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(f)], check=True, capture_output=True,
                              text=True).stdout
        for line in text.splitlines():
            key, _, value = line.strip().lstrip("- ").partition(":")
            if key == ".agpr_count":          # first field of a kernel
                cur = {}
            cur[key] = value.strip()
            if key == ".name" and "emit_kernel" in value:
                kernels[value.strip()] = cur
    return kernels


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("tile", [8, 16, 32, 64])
@pytest.mark.parametrize("profile", [0, 1])
def test_plain_bunch_kernels_use_no_scratch(notes, precision, tile, profile):
    k = notes[f"_ZN3ckv11emit_kernelILi{precision}ELi{tile}ELi{profile}EEEvNS_4ArgsE"]
    assert int(k[".private_segment_fixed_size"]) == 0
    assert int(k[".vgpr_spill_count"]) == 0
    assert int(k[".vgpr_count"]) <= 128
