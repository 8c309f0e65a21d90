"""Rows of map words by reciprocal (csrc/cb_claim.h, map_row), compiled for the host and compared with divisions over every size of map whose list is extracted in
the launch of detection: up to 2^17 words, rows of up to 2^11."""
import ctypes as C
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1808_05488_amd", "csrc")

SOURCE = r"""
#include "cb_claim.h"
extern "C" int first_wrong(unsigned w, unsigned words)
{
    const unsigned inv = cb::map_row_inv(w);
    for (unsigned it = 0; it < words; ++it)
        if (cb::map_row(it, inv) != it / w) return (int)it;
    return -1;
}
"""


def test_rows_are_those_of_the_division(tmp_path):
    src, lib = tmp_path / "rows.cpp", tmp_path / "librows.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    rows = C.CDLL(str(lib))
    for w in (*range(1, 70), 100, 127, 128, 129, 255, 1000, 1023, 1024, 2047, 2048):
        assert rows.first_wrong(w, 1 << 17) == -1, w
