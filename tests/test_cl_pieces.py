"""Taps and channels of the channel-last kernel's 16-byte pieces (csrc/cb_cl_rules.h), compiled for the host and compared with divisions,
over every number of channels that is a whole number of pieces and up to the kernel's longest filter."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1808_05488_amd", "csrc")

SOURCE = r"""
#include "cb_cl_rules.h"
// first piece that disagrees (value * 4 + error), or -1; stages begin at multiples of 32 values, pieces every 4, a few stages run past the filter
extern "C" long pieces(int Cs, int kmax, int stage)
{
    const cb::ClDiv d = cb::cl_div(640, 480, 3, Cs);
    for (unsigned kb = 0; kb < (unsigned)kmax + 4u * stage; kb += stage)
        for (unsigned o = 0; o < (unsigned)stage; o += 4) {
            const unsigned dt = cb::cl_tap(d, o), cl = o - dt * Cs;
            if (dt != o / Cs) return (long)o * 4 + 1;
            unsigned tap, coff;
            cb::cl_piece(d, Cs, kb, dt, cl, tap, coff);
            if (tap != (kb + o) / Cs || coff + cl != (kb + o) % Cs) return (long)(kb + o) * 4 + 2;
            if (cb::cl_tap(d, kb + o) != (kb + o) / Cs) return (long)(kb + o) * 4 + 3;
        }
    return -1;
}
extern "C" unsigned split(int f32, int N, int O, unsigned nkg, unsigned ws)
{
    return f32 ? cb::cl_split<true>(N, O, nkg, ws) : cb::cl_split<false>(N, O, nkg, ws);
}
extern "C" int fits(int Cs, int taps) { return cb::cl_fits(Cs, taps); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("cl_pieces")
    src, lib = d / "pieces.cpp", d / "libpieces.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    lib = C.CDLL(str(lib))
    lib.pieces.restype = C.c_long
    return lib


def test_tap_and_channel_of_every_piece(rules):
    for cs in list(range(4, 800, 4)) + list(range(800, 32768, 1012)) + [32764, 32768]:
        for stage in (32, 64, 512):
            assert rules.pieces(cs, 65536, stage) == -1, (cs, stage)


def test_longest_filter(rules):
    assert rules.fits(32768, 2) and rules.fits(4, 961) and rules.fits(68, 961)
    assert not rules.fits(32772, 1) and not rules.fits(72, 961) and not rules.fits(32768, 3)


def test_parts_of_k_fit_what_they_need(rules):
    """Every choice leaves each part eight groups of K, its partial sums in the workspace and its tiles in the counters; none without a workspace."""
    rules.split.restype = C.c_uint
    chosen = set()
    for f32 in (0, 1):
        for o in (100, 128, 256, 300, 512, 2000):
            for nkg in (96, 98, 144, 256, 392, 2048):
                for n in (1, 31, 32, 33, 500, 1054, 2184, 5000, 8193, 40000, 1 << 22):
                    assert rules.split(f32, n, o, nkg, 0) == 0
                    for ws in (1 << 16, 1 << 20, 16 << 20):
                        r = rules.split(f32, n, o, nkg, ws)
                        if not r:
                            continue
                        parts, bn = r & 15, 64 if r & 16 else 32
                        tiles = -(-n // bn) * -(-o // 128)
                        chosen.add((parts, bn))
                        assert 2 <= parts <= 8 and -(-nkg // parts) >= 8 and tiles <= 256 and tiles * parts * 128 * bn * 4 <= ws
    assert {bn for _, bn in chosen} == {32, 64} and len(chosen) >= 8
