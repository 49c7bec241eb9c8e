"""No kernel of the library keeps anything in scratch memory: not a register spilled, no array indexed at run time.  Read off the
metadata of the library's own code objects; no GPU involved."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2508_00441_amd import binding

LLVM = "/opt/rocm/llvm/bin/"


@pytest.mark.skipif(not os.path.exists(LLVM + "llvm-readelf"), reason="no LLVM tools")
def test_kernels_use_no_scratch(tmp_path):
    lib = tmp_path / "lib.so"
    shutil.copy(binding.LIB_PATH, lib)
    subprocess.check_call([LLVM + "llvm-objdump", "--offloading", str(lib)], cwd=tmp_path, stdout=subprocess.DEVNULL)
    kernels, spilling = 0, []
    for f in sorted(tmp_path.glob("*gfx950*")):
        notes = subprocess.check_output([LLVM + "llvm-readelf", "--notes", str(f)], text=True)
        for part in re.split(r"^  - \.agpr_count", notes, flags=re.M)[1:]:
            name = re.search(r"^    \.name: +(\S+)", part, flags=re.M).group(1)
            scratch, spills = (int(re.search(rf"^    \.{key}: +(\d+)", part, flags=re.M).group(1)) for key in ("private_segment_fixed_size", "vgpr_spill_count"))
            kernels += 1
            if scratch or spills:
                spilling.append((name, scratch, spills))
    assert kernels > 80
    assert not spilling, spilling
