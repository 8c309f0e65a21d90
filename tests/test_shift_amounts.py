"""No kernel takes the amount of a 64-bit shift from the last vector register of its allocation (registers come in eights).  gfx950 now
and then reads register 0 instead: the compiler avoids the form for gfx90a, whose bug it is known as, and not here.  Seen as change lists
that missed or moved a few pixels in one frame of twenty; the kernels' code is checked, since tests of results rarely show it."""
import glob
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_1808_05488_amd import build


def _shifts(path):
    """(kernel, instruction) of every such shift in the code of one source file, and the number of 64-bit shifts by a register."""
    r = subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", path, "-o", "-"], check=True, capture_output=True, text=True)
    regs, kernel = {}, None
    for line in r.stdout.splitlines():
        m = re.match(r"\s*\.amdhsa_(kernel|next_free_vgpr) (\S+)", line)
        if m and m.group(1) == "kernel":
            kernel = m.group(2)
        elif m:
            regs[kernel] = (int(m.group(2)) + 7) // 8 * 8
    found, n, kernel = [], 0, None
    for line in r.stdout.splitlines():
        m = re.match(r"^(_Z\S+):", line)
        if m:
            kernel = m.group(1)
        m = re.match(r"\s+v_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\S* v\[\d+:\d+\], v(\d+),", line)
        if m:
            n += 1
            if int(m.group(1)) == regs[kernel] - 1:
                found.append((kernel, line.strip()))
    return found, n


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_no_64_bit_shift_by_the_last_register():
    files = sorted(glob.glob(os.path.join(build.CSRC, "*.hip")))
    with ThreadPoolExecutor(max_workers=8) as ex:
        results = list(ex.map(_shifts, files))
    assert sum(n for _, n in results) > 100          # the pattern still matches what the compiler writes
    assert [f for found, _ in results for f in found] == []
