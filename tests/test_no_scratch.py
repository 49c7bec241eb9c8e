"""No kernel of the library keeps anything in scratch memory: not a register spilled, no array indexed at run time.  Read off the
metadata of the library's own code objects; no GPU involved."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2508_00441_amd import binding

LLVM = "/opt/rocm/llvm/bin/"


def _kernel_notes(tmp_path):
    """(name, the metadata lines) of every kernel in the library."""
    lib = tmp_path / "lib.so"
    shutil.copy(binding.LIB_PATH, lib)
    subprocess.check_call([LLVM + "llvm-objdump", "--offloading", str(lib)], cwd=tmp_path, stdout=subprocess.DEVNULL)
    for f in sorted(tmp_path.glob("*gfx950*")):
        notes = subprocess.check_output([LLVM + "llvm-readelf", "--notes", str(f)], text=True)
        for part in re.split(r"^  - \.agpr_count", notes, flags=re.M)[1:]:
            yield re.search(r"^    \.name: +(\S+)", part, flags=re.M).group(1), part


def _value(part, key):
    return int(re.search(rf"^    \.{key}: +(\d+)", part, flags=re.M).group(1))


@pytest.mark.skipif(not os.path.exists(LLVM + "llvm-readelf"), reason="no LLVM tools")
def test_kernels_use_no_scratch(tmp_path):
    kernels, spilling = 0, []
    for name, part in _kernel_notes(tmp_path):
        scratch, spills = _value(part, "private_segment_fixed_size"), _value(part, "vgpr_spill_count")
        kernels += 1
        if scratch or spills:
            spilling.append((name, scratch, spills))
    assert kernels > 80
    assert not spilling, spilling


@pytest.mark.skipif(not os.path.exists(LLVM + "llvm-readelf"), reason="no LLVM tools")
def test_the_one_pass_with_few_slices_leaves_room_for_two_workgroups(tmp_path):
    """ladder_sums_kernel<FMT, S, MODE, PART> with S <= 8: half the registers and less than half the LDS of a compute unit."""
    seen = 0
    for name, part in _kernel_notes(tmp_path):
        m = re.search(r"ladder_sums_kernelILi\d+ELi(\d+)ELi", name)
        if m and int(m.group(1)) <= 8:
            seen += 1
            assert _value(part, "vgpr_count") <= 256 and 2 * _value(part, "group_segment_fixed_size") <= 160 * 1024, name
    assert seen >= 30
