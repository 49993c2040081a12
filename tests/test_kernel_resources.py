"""Registers and placement of the built bunch kernels (CPU: the code objects' own notes and
symbols).

The plain bunch kernels hold their state in the 128 vector registers that 16 waves leave
a lane: no scratch, no spilled vector register.  The functions that walk a ray through the
cells start on an instruction cache line."""
import os
import shutil
import subprocess

import pytest

from paper_2006_14927_amd import ckv

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    if not os.path.exists(ckv.LIB_PATH) or not os.path.exists(f"{LLVM}/llvm-objdump"):
        pytest.skip("needs the built library and llvm-objdump")
    d = tmp_path_factory.mktemp("co")
    shutil.copy(ckv.LIB_PATH, d / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    return sorted(d.glob("lib.so.*gfx950"))


@pytest.fixture(scope="module")
def notes(code_objects):
    kernels, cur = {}, {}
    for f in code_objects:
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


def test_ray_walks_start_on_a_cache_line(code_objects):
    found = {}
    for f in code_objects:
        text = subprocess.run([f"{LLVM}/llvm-readelf", "-s", str(f)], check=True, capture_output=True, text=True).stdout
        for line in text.splitlines():
            if " FUNC " in line and ("propagate_curved_call" in line or "propagate_exact_call" in line):
                found[f.name, line.split()[-1]] = int(line.split()[1], 16)
    assert len(found) >= 2
    assert all(at % 64 == 0 for at in found.values()), found
