"""float32 sums of the widest tiles of the channel-last kernel (csrc/cb_fused_cl.h), whole and with K in parts, against float64: operands keep all 24 bits, so that a filter whose
only weight is 1 gives its input back bit for bit and sums of one or two products have float32's own rounding; dense sums of any range of values err as one chain of products does."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest
import torch

if torch.cuda.is_available():
    import paper_1808_05488_amd as cb

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1808_05488_amd", "csrc")

SOURCE = r"""
#include "cb_cl_rules.h"
template <int SHAPE> int tile(int N, int O, int Cs, int taps)
{
    int t = -1;
    cb::cl_tile<true, SHAPE>(N, O, Cs, taps, Cs * taps, [&](auto x) { t = decltype(x)::value; });
    return t;
}
// instance * 1000 + tile, or 200 000 + what cl_split says of a layer whose K is divided
extern "C" int full_update(int C, int O, int k, int H, int W)
{
    const int N = H * W, taps = k * k;
    const unsigned nkg = ((unsigned)(C * taps) + 31u) / 32u;
    if (cb::cl_shape(O, N, true) == 128 && cb::cl_filter_kb(O, nkg, true) >= cb::CL_FAR_KB && cb::cl_split_pays(nkg, true))
        if (const unsigned s = cb::cl_split<true>(N, O, nkg, 16u << 20)) return 200000 + (int)s;
    switch (cb::cl_shape(O, N, true)) {
        case 32: return 32000 + tile<32>(N, O, C, taps);
        case 64: return 64000 + tile<64>(N, O, C, taps);
        default: return 128000 + tile<128>(N, O, C, taps);
    }
}
"""

# what runs the full update (as above), input channels, output channels, filter size, height, width
TILES = [
    (32003, 16, 24, 3, 133, 143),        # 32 x 128
    (64003, 16, 45, 3, 91, 99),          # 64 x 64, the last row tile in part
    (64003, 64, 64, 3, 480, 640),
    (128003, 48, 96, 5, 90, 93),         # 128 x 32, channels that are no power of two
    (128003, 256, 130, 3, 60, 61),
    (128004, 32, 72, 3, 91, 99),         # 128 x 64
    (128004, 288, 96, 1, 92, 164),
    (200000 + 16 + 2, 512, 512, 3, 46, 82),     # 128 x 64, two parts of K
    (200003, 256, 128, 9, 60, 80),       # 128 x 32, three
]


def test_layers_run_the_tiles_they_stand_for(tmp_path):
    src, lib = tmp_path / "wide.cpp", tmp_path / "libwide.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    rules = C.CDLL(str(lib))
    for what, *geom in TILES:
        assert rules.full_update(*geom) == what, geom


def conv64(x, w):
    o, c, k, _ = w.shape
    h, wd = x.shape[1:]
    xp = torch.nn.functional.pad(x.double(), (k // 2,) * 4)
    y = torch.zeros((o, h * wd), dtype=torch.float64, device=x.device)
    for j in range(k):
        for i in range(k):
            y.addmm_(w[:, :, j, i].double().contiguous(), xp[:, j:j + h, i:i + wd].reshape(c, -1))
    return y.view(o, h, wd)


def full_update(x, w):
    return cb.Layer(w, None, 1, w.shape[2] // 2, x.shape[1], x.shape[2], False).process_frame(x, 0.0)


def generator(*seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(hash(seed) & 0xFFFFFFF)
    return g


@pytest.mark.gpu
@pytest.mark.parametrize("tile", TILES)
def test_single_weights_pass_their_input_on(tile):
    what, ci, co, k, H, W = tile
    print("single weights", tile, flush=True)
    g = generator(*tile)
    x = (torch.rand((ci, H, W), generator=g, device="cuda") * 2 - 1) * torch.exp2(torch.randint(-30, 30, (ci, H, W), generator=g, device="cuda").float())
    w = torch.zeros((co, ci, k, k), device="cuda")
    o = torch.arange(co, device="cuda")
    w[o, o * 7 % ci, k // 2, k // 2] = 1
    assert torch.equal(full_update(x, w), x[o * 7 % ci])


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 2])
@pytest.mark.parametrize("side", ["pixels", "weights"])
@pytest.mark.parametrize("tile", TILES)
def test_sums_of_few_products(tile, side, n):
    """One product: a rounding of the sum, 2^-24 / sqrt(3) of it in the mean.  Two: the first is rounded once for each of the instructions that add the second's terms."""
    what, ci, co, k, H, W = tile
    print("few products", tile, side, n, flush=True)
    g = generator(*tile, n)
    x = torch.rand((ci, H, W), generator=g, device="cuda")
    w = torch.randn((co, ci, k, k), generator=g, device="cuda")
    if side == "pixels":                 # every filter position sees one pixel, n channels of it
        on = torch.zeros_like(x)
        on.scatter_(0, torch.rand((ci, H, W), generator=g, device="cuda").topk(n, 0).indices, 1.0)
        grid = torch.zeros((H, W), device="cuda")
        grid[::k, ::k] = 1
        x = x * on * grid
    else:
        on = torch.zeros((co, ci * k * k), device="cuda")
        on.scatter_(1, torch.rand(on.shape, generator=g, device="cuda").topk(n, 1).indices, 1.0)
        w = w * on.view_as(w)
    y, ref = full_update(x, w).double(), conv64(x, w)
    assert ((y - ref).norm() / ref.norm()).item() < {1: 3.9e-8, 2: 6e-8}[n]


KINDS = ["ordinary", "wide pixels", "wide weights", "both wide", "large where weights are zero", "large weights where pixels are zero", "dark columns", "first taps small"]


@pytest.mark.gpu
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("tile", TILES)
def test_any_range_of_values(tile, kind):
    what, ci, co, k, H, W = tile
    print("any range", tile, kind, flush=True)
    rng = np.random.default_rng(ci + co + len(kind))

    def wide(shape, lo, hi):
        return (rng.uniform(-1, 1, shape) * 2.0 ** rng.uniform(lo, hi, shape)).astype(np.float32)

    x = rng.uniform(-1, 1, (ci, H, W)).astype(np.float32)
    w = (rng.standard_normal((co, ci, k, k)) / (ci * k * k) ** 0.5).astype(np.float32)
    if kind in ("wide pixels", "both wide"):
        x = wide((ci, H, W), -60, 12)
        x[rng.random((ci, H, W)) < 0.5] = 0
    if kind in ("wide weights", "both wide"):
        w = wide(w.shape, -60, 12)
        w[rng.random(w.shape) < 0.5] = 0
    if kind == "large where weights are zero":       # the sums are those of the small channels alone
        x[::2] *= np.float32(2.0 ** 9)
        x[1::2] *= np.float32(2.0 ** -25)
        w[:, ::2] = 0
    if kind == "large weights where pixels are zero":
        w[:, ::2] *= np.float32(2.0 ** 10)
        w[:, 1::2] *= np.float32(2.0 ** -30)
        x[::2] = 0
    if kind == "dark columns":                        # most of the image at 2^-30, a bright region within reach of some filters
        x *= np.float32(2.0 ** -30)
        x[:, H // 3:H // 2, W // 3:W // 2] *= np.float32(2.0 ** 36)
    if kind == "first taps small":
        x[:, ::2] *= np.float32(2.0 ** -16)
    x, w = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y, ref, mag = full_update(x, w).double(), conv64(x, w), conv64(x.abs(), w.abs())
    K = ci * k * k
    assert torch.isfinite(y).all()
    # every instruction (six for 32 products) rounds the partial sum, and what it adds, by at most 2^-24 of the magnitudes
    bad = (y - ref).abs() > (12 * (K / 32 + 1) + 8) * 2.0 ** -24 * mag + 2.0 ** -149
    assert not bad.any(), int(bad.sum())
    if kind == "ordinary":
        # the roundings of one chain, 2^-24 / sqrt(3) of partial sums that grow from zero: sqrt(6 K / 32 / 6) in the mean; twice that
        assert ((y - ref).norm() / ref.norm()).item() < 2.0 ** -24 * (K / 8 + 4) ** 0.5
