"""What the compiler makes of change detection's cache hints.  The frame is read once and, where a state does not fit the
last-level cache, so is the state: both loads carry the non-temporal mark.  Of two loads of the same type and address in the two arms
of a condition the compiler makes one without the mark, which shows in no result, only in time."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1808_05488_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_state_loads_past_the_cache_are_marked(tmp_path):
    asm = tmp_path / "detect.s"
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "cb_detect.hip"), "-o", str(asm)],
                   check=True, capture_output=True)
    marked, kernel = {}, None
    for line in asm.read_text().splitlines():
        m = re.match(r"^_ZN2cb\S*detect_reg_kernelI([tf])Li(\d+)ELi\d+ELi(\d+)ELi\d+ELb[01]EE\S*:", line)
        if m:
            kernel = line
            marked[kernel] = [m.group(1), int(m.group(2)), int(m.group(3)), 0]
        elif line.startswith(".Lfunc_end"):
            kernel = None
        elif kernel and re.search(r"global_load_\w+.*\bnt\b", line):
            marked[kernel][3] += 1
    wide = [v for v in marked.values() if v[1] == 4]
    assert {v[0] for v in wide} == {"t", "f"} and len(wide) >= 16
    for dtype, _, channels, n in wide:               # per lane: each channel of the frame and of the state
        assert n >= 2 * channels, (dtype, channels, n)
