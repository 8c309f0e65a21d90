"""float32 layers on the wide tiles of the channel-last kernel (csrc/cb_fused_cl.h): values over far more than float16's range, with zeros where the large ones would hide what
the small ones lost, against float64, element by element, and errors of whole layers."""
import numpy as np
import pytest
import torch

if torch.cuda.is_available():
    import paper_1808_05488_amd as cb

# (input channels, output channels, filter size, height, width): full updates on 32 x 128, 64 x 64, 128 x 32, 128 x 64 tiles, whole and in parts of K, channels that are no power of two
GEOMS = [(16, 24, 3, 133, 143), (16, 45, 3, 91, 99), (64, 64, 3, 143, 141), (24, 72, 3, 75, 81), (32, 72, 3, 91, 99), (48, 96, 5, 90, 93), (256, 130, 3, 60, 61), (512, 512, 3, 46, 82)]
KINDS = ["ordinary", "wide pixels", "wide weights", "both wide", "large where weights are zero", "large weights where pixels are zero", "dark columns", "first taps small"]


@pytest.mark.gpu
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("geom", GEOMS)
def test_any_range_of_values(geom, kind):
    ci, co, k, H, W = geom
    print("half terms", geom, kind, flush=True)
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
    if kind == "first taps small":                    # the rest of a column outgrows its scale
        x[:, ::2] *= np.float32(2.0 ** -16)
    b = np.zeros(co, np.float32)
    y = cb.Layer(torch.from_numpy(w).cuda(), torch.from_numpy(b).cuda(), 1, k // 2, H, W, False).process_frame(torch.from_numpy(x).cuda(), 0.0).double().cpu()
    xt, wt = torch.from_numpy(x)[None].double(), torch.from_numpy(w).double()
    ref = torch.nn.functional.conv2d(xt, wt, None, 1, k // 2)[0]
    mag = torch.nn.functional.conv2d(xt.abs(), wt.abs(), None, 1, k // 2)[0]
    # terms: 2^-22 of either factor, what is lost below them 2^-22 of the sum; the sum rounded at most once a product
    bound = (ci * k * k + 16) * 2.0 ** -24 * mag + 2.0 ** -149
    assert torch.isfinite(y).all()
    bad = (y - ref).abs() > bound
    assert not bad.any(), (int(bad.sum()), ((y - ref).abs() / bound).max().item())


@pytest.mark.gpu
@pytest.mark.parametrize("geom", [(64, 64, 3, 143, 141), (256, 100, 3, 61, 67), (48, 96, 5, 143, 141)])
def test_errors_are_no_larger_than_those_of_six_products(geom):
    """Relative 2-norm errors of whole layers against float64, positive and signed inputs: below those measured with one chain of six bfloat16 products (7.3e-7, 5.2e-7) and the
    two-chain tile's (1.4e-7)."""
    ci, co, k, H, W = geom
    limit = {64: 1.5e-7, 256: 4e-7, 48: 3e-7}[ci]
    g = torch.Generator(device="cuda")
    g.manual_seed(ci)
    for signed in (False, True):
        x = torch.randn((ci, H, W), generator=g, device="cuda") if signed else torch.rand((ci, H, W), generator=g, device="cuda")
        w = torch.randn((co, ci, k, k), generator=g, device="cuda") * (2.0 / (ci * k * k)) ** 0.5
        y = cb.Layer(w, None, 1, k // 2, H, W, False).process_frame(x, 0.0).double().cpu()
        ref = torch.nn.functional.conv2d(x.cpu()[None].double(), w.cpu().double(), None, 1, k // 2)[0]
        assert ((y - ref).norm() / ref.norm()).item() < limit
