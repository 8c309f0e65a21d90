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
