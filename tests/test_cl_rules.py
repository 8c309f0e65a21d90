"""Rules of the channel-last fused kernel that are plain arithmetic (csrc/cb_cl_rules.h), compiled for the host and
compared with their definitions."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1808_05488_amd", "csrc")

SOURCE = r"""
#include "cb_cl_rules.h"
extern "C" int row(int q, int Wo, int Ho, int kw) { return cb::cl_row(cb::cl_div(Wo, Ho, kw), q, Wo); }
extern "C" unsigned inv_kw(int kw) { return cb::cl_div(1, 1, kw).inv_kw; }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("cl_rules")
    src, lib = d / "rules.cpp", d / "librules.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    return C.CDLL(str(lib))


# Output maps of fewer than 2^30 pixels: narrow and tall (the product of the reciprocal reaches 2^64 at row 2^22), and wide.
@pytest.mark.parametrize("Wo", [1, 2, 3, 4, 7, 63, 255, 256, 640, 1921, 4095, 4096, 5000, 1 << 20])
def test_output_row_of_a_listed_pixel(rules, Wo):
    top = ((1 << 30) - 1) // Wo
    for Ho in {1, min(top, 1000), min(top, (1 << 22) - 1), min(top, 1 << 22), min(top, (1 << 22) + 1), min(top, 5000000), top}:
        rows = {0, 1, Ho // 3, Ho // 2, Ho - 2, Ho - 1} | {(1 << 22) + d for d in (-2, -1, 0, 1)}
        for y in sorted(r for r in rows if 0 <= r < Ho):
            for x in {0, Wo // 2, Wo - 1}:
                q = y * Wo + x
                assert rules.row(q, Wo, Ho, 3) == y, (Wo, Ho, q)


def test_filter_row_of_a_tap(rules):
    """Every tap of every filter the kernel takes, and the taps that pad K and run ahead of it (a few stages of 64)."""
    for kw in range(1, 32):
        inv = rules.inv_kw(kw)
        for tap in range(31 * kw + 256):
            assert (tap * inv) >> 16 == tap // kw, (kw, tap)
