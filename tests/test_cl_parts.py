"""Layers whose filters are divided (csrc/cb_cl_rules.h), compiled for the host: float32 K is divided only where the sums round no
worse than those of the tile that would take all of K, and the items of a layer come out even enough among the XCDs."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1808_05488_amd", "csrc")

SOURCE = r"""
#include "cb_cl_rules.h"
extern "C" unsigned split(int N, int O, unsigned nkg, unsigned ws) { return cb::cl_split<true>(N, O, nkg, ws); }
extern "C" int far(int O, unsigned nkg) { return cb::cl_filter_kb(O, nkg, true) >= cb::CL_FAR_KB; }
extern "C" unsigned rows(unsigned MT, unsigned NT, unsigned parts, unsigned filter_kb, unsigned pixel_kb) { return cb::cl_xcd_rows(MT, NT, parts, filter_kb, pixel_kb); }
extern "C" int tile(int N, int O, int C, int taps)
{
    int t = -1;
    cb::cl_tile<true, 128>(N, O, C, taps, C * taps, [&](auto x) { t = decltype(x)::value; });
    return t;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("cl_parts")
    src, lib = d / "parts.cpp", d / "libparts.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    lib = C.CDLL(str(lib))
    lib.split.restype = C.c_uint
    return lib


def test_divided_sums_round_no_worse(rules):
    """A chain of sums over K errs like sqrt(K) * its partial sums, so p parts err 1 / sqrt(p) of one; a chain of their own for the small terms
    takes 0.39 of it (measured: 4.1e-7 of 1.06e-6 at K = 4 608), four wavefronts that share K half of that."""
    one, two, four = 1.0, 0.39, 0.195
    whole = {0: four, 1: two, 2: two, 3: one, 4: one}       # 16 x 16, 64 x 16, 64 x 32, 128 x 32, 128 x 64
    divided = set()
    for o in (65, 100, 128, 200, 256, 260, 384, 450, 512, 640, 1024):
        for c, taps in ((512, 9), (64, 49), (128, 81), (256, 81), (128, 25), (1024, 9), (2048, 1)):
            nkg = -(-c * taps // 32)
            if nkg < 96 or not rules.far(o, nkg):                # (K is not divided)
                continue
            for n in (*range(1, 400, 7), *range(400, 8000, 61), 20000):
                r = rules.split(n, o, nkg, 16 << 20)
                if not r:
                    continue
                t = rules.tile(n, o, c, taps)
                parts = r & 15
                err = (one if r & 16 else two) / parts ** 0.5
                divided.add((t, bool(r & 16)))
                assert err <= whole[t] * 1.001, (n, o, c, taps, t, r)
    assert len(divided) >= 4


def test_no_xcd_has_much_more_than_its_share(rules):
    """Items of every XCD counted one by one as the kernel walks them: all of them once, and the most on one XCD at most an eighth above what undivided
    rows give it, or no more than its 32 compute units."""
    def items(mt, nt, l):
        per, cols = (mt + (1 << l) - 1) >> l, (nt + (8 >> l) - 1) >> (3 - l)
        on = []
        for x in range(8):
            m0, c0 = (x & ((1 << l) - 1)) * per, (x >> l) * cols
            on.append({(m, c) for m in range(m0, min(m0 + per, mt)) for c in range(c0, min(c0 + cols, nt))})
        return on

    seen = set()
    for mt in (1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 17, 20, 33):
        for nt in (1, 2, 3, 7, 8, 9, 15, 16, 18, 23, 36, 59, 62, 118, 150, 236):
            for parts in (1, 2, 5, 8):
                for filter_kb, pixel_kb in ((4096, 100), (4096, 700), (4096, 2000), (4096, 9000)):
                    l = rules.rows(mt, nt, parts, filter_kb, pixel_kb)
                    on = items(mt, nt, l)
                    assert sum(len(s) for s in on) == mt * nt and len(set().union(*on)) == mt * nt
                    most, whole = (max(len(s) for s in o) for o in (on, items(mt, nt, 0)))
                    assert most * 8 <= whole * 9 or most * parts <= 32, (mt, nt, parts, l)
                    seen.add(l)
    assert seen == {0, 1, 2, 3}
