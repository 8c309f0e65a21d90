"""Rules of the channel-last fused kernel that are plain arithmetic (csrc/cb_cl_rules.h), compiled for the host and
compared with their definitions."""
import ctypes as C
import os
import subprocess

import pytest

from cl_tiles import LARGE_MAP_LAYER, LARGE_MAP_REGIONS, TILE_CASES

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1808_05488_amd", "csrc")

SOURCE = r"""
#include "cb_cl_rules.h"
extern "C" int row(int q, int Wo, int Ho, int kw) { return cb::cl_row(cb::cl_div(Wo, Ho, kw), q, Wo); }
extern "C" unsigned inv_kw(int kw) { return cb::cl_div(1, 1, kw).inv_kw; }
template <bool F32> int tile(int N, int O, int Po, int Cs, int taps, int R)
{
    int t = -1;
    auto run = [&](auto tile) { t = decltype(tile)::value; };
    switch (cb::cl_shape(O, Po, F32)) {
        case 16: cb::cl_tile<F32, 16>(N, O, Cs, taps, R, run); break;
        case 32: cb::cl_tile<F32, 32>(N, O, Cs, taps, R, run); break;
        case 64: cb::cl_tile<F32, 64>(N, O, Cs, taps, R, run); break;
        case 129: cb::cl_tile<F32, 129>(N, O, Cs, taps, R, run); break;
        default: cb::cl_tile<F32, 128>(N, O, Cs, taps, R, run);
    }
    return t;
}
extern "C" int tile(int bf16, int N, int O, int Po, int Cs, int taps, int R)
{
    return bf16 ? tile<false>(N, O, Po, Cs, taps, R) : tile<true>(N, O, Po, Cs, taps, R);
}
extern "C" int shape(int O, int Po, int bf16) { return cb::cl_shape(O, Po, !bf16); }
extern "C" int tiles(int shape) { return cb::cl_tiles(shape); }
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


def test_tile_cases_cover_every_tile(rules):
    """Each layer picks the tile it stands for, and together they pick every tile of every instance: a change of the rule
    that moves one shows up here."""
    for shape, tile, bf16, c, o, k, h, w in TILE_CASES:
        pixel = 16 // (2 if bf16 else 4)
        cs = pixel if c <= pixel else c
        assert rules.shape(o, h * w, bf16) == shape
        assert rules.tile(bf16, h * w, o, h * w, cs, k * k, c * k * k) == tile, (shape, tile, bf16, c, o, k, h, w)
    c, o, k, h, w = LARGE_MAP_LAYER
    large = rules.shape(o, h * w, True)
    for side, tile in LARGE_MAP_REGIONS:
        assert rules.tile(True, (side + k - 1) ** 2, o, h * w, c, k * k, c * k * k) == tile, (side, tile)
    every = {(s, t, b) for s in (16, 32, 64, 128) for b in (False, True) for t in range(rules.tiles(s))}
    every |= {(129, t, True) for t in range(rules.tiles(129))}
    assert {(s, t, b) for s, t, b, *_ in TILE_CASES} | {(large, t, True) for _, t in LARGE_MAP_REGIONS} == every


@pytest.mark.parametrize("c,o,n,tile", [(512, 512, 1425, 2), (512, 512, 1300, 2), (256, 512, 1425, 3)])
def test_medium_counts_with_short_and_long_filters(rules, c, o, n, tile):
    """bfloat16, 3x3, 46x82: between one round of 128 x 32 tiles and two of 64 x 32 ones."""
    assert rules.tile(True, n, o, 46 * 82, c, 9, 9 * c) == tile
