"""The instructions of the built library's kernels (a listing of the library built here, on the CPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_10233_amd import binding, build_lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# a 64-bit vector shift whose amount is a vector register
SHIFT = re.compile(r"v_(?:lshlrev|lshrrev|ashrrev)_(?:b64|i64)\S*\s+v\[\d+:\d+\], v\d+,")


def listing(lib, folder):
    """Disassembly of every gfx950 code object of the library."""
    copy = shutil.copy(lib, folder)
    subprocess.run([OBJDUMP, "--offloading", os.path.basename(copy)], cwd=folder, check=True, capture_output=True)
    objects = sorted(f for f in os.listdir(folder) if f.endswith("gfx950") and os.path.getsize(os.path.join(folder, f)))
    assert objects
    return [subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(folder, f)], check=True, capture_output=True,
                           text=True).stdout for f in objects]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_64_bit_shift_by_a_lanes_amount(tmp_path):
    """Such a shift takes another amount in some waves when its amount register is the last of the kernel's
    allocation (dev.h, shl32), which any edit can bring about: no kernel may hold one."""
    if not os.path.exists(binding.lib_path()):
        build_lib.build()
    kernels, found = 0, []
    for text in listing(binding.lib_path(), str(tmp_path)):
        name = ""
        for line in text.splitlines():
            if line.endswith(">:"):
                name = line.split("<")[-1][:-2]
                kernels += 1
            elif SHIFT.search(line):
                found.append((name, line.strip()))
    assert kernels > 100
    assert not found, "%d in %s" % (len(found), sorted({k for k, _ in found})[:8])
