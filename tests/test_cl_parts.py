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
// the tile of 128-row layers from costs in 64 bits
extern "C" int tile64(int f32, int N, int O, unsigned nkg)
{
    auto cost = [&](int bm, int bn, long long a0, long long a1, long long a2, long long a3, long long b0, long long b1, long long b2, long long b3) {
        const long long tiles = ((N + bn - 1LL) / bn) * ((O + bm - 1LL) / bm), l0 = f32 ? a0 : b0, l1 = f32 ? a1 : b1, c0 = f32 ? a2 : b2, c1 = f32 ? a3 : b3;
        const long long lat = l0 + l1 * nkg, busy = (tiles + 255) / 256 * (c0 + c1 * nkg);
        return busy > lat ? busy : lat;
    };
    const bool far = f32 && (long long)O * nkg * 32 > 700000;
    const long long v[5] = {cost(16, 16, 100, 94, 1260, far ? 80 : 49, 200, 30, 870, 16), cost(64, 16, 0, 176, 1250, 120, 100, 58, 650, 41),
                            cost(64, 32, 1000, 300, 1400, 203, 400, 80, 1100, 47), cost(128, 32, 1800, 380, 1000, 320, 1500, 100, 100, 96),
                            cost(128, 64, 900, 745, 2900, 510, 2000, 190, 1000, 140)};
    int best = 0;
    for (int i = 1; i < 5; ++i) if (v[i] < v[best]) best = i;
    return best;
}
extern "C" int tile_bf16(int N, int O, int C, int taps)
{
    int t = -1;
    cb::cl_tile<false, 128>(N, O, C, taps, C * taps, [&](auto x) { t = decltype(x)::value; });
    return t;
}
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


def test_costs_of_the_largest_layers(rules):
    """The tile picked with costs in 32 bits is the one of 64 bits, up to the longest filters and the most listed pixels."""
    for o in (65, 100, 128, 256, 500, 1024, 2048, 30000, (1 << 20) - 1):
        for c, taps in ((32, 9), (512, 9), (1024, 49), (8192, 8), (32768, 2), (65536 // 25 // 4 * 4, 25)):
            for n in (1000, 307200, 2073600, 8294400, 100000000, (1 << 30) - 1):
                for f32, pick in ((1, rules.tile), (0, rules.tile_bf16)):
                    assert pick(n, o, c, taps) == rules.tile64(f32, n, o, (c * taps + 31) // 32), (n, o, c, taps, f32)
