"""The bound that the GPU tests put on the float32 error of split products tells a full set of products from one with a
term left out.  The products are restated here with torch's bfloat16 rounding and summed in float64, so that only
what the split and the choice of products lose remains."""
import pytest
import torch

from parity import split_bound


def terms(x):
    out = []
    for _ in range(3):
        t = x.to(torch.bfloat16).to(torch.float32)
        out.append(t.double())
        x = x - t
    return out, x


@pytest.mark.parametrize("K", [576, 2304])
def test_bound_tells_a_missing_term(K):
    g = torch.Generator()
    g.manual_seed(K)
    a, b = torch.randn((200, K), generator=g), torch.randn((K, 150), generator=g)
    (ah, am, al), ra = terms(a)
    (bh, bm, bl), rb = terms(b)
    assert not ra.any() and not rb.any()                  # three terms are the whole value
    ref = a.double() @ b.double()

    def err(y):
        return ((y - ref).norm() / ref.norm()).item()

    four = ah @ bh + ah @ bm + am @ bh + am @ bm
    six = four + ah @ bl + al @ bh
    assert err(six) < 0.1 * split_bound(K)
    assert err(four) > split_bound(K)                     # without h*l and l*h
    assert err(ah @ bh + ah @ bm + am @ bh) > split_bound(K)
    assert err(six - am @ bm) > split_bound(K)


@pytest.mark.parametrize("e", [-140, -126, -110, 0, 100])
def test_split_of_scaled_values_is_exact(e):
    """... over the whole range of float32 with 2^24 in front, which keeps the last term of the smallest numbers inside bfloat16's
    normal range; as they are, values below about 2^-110 lose theirs."""
    g = torch.Generator()
    g.manual_seed(3)
    x = ((torch.rand(20000, generator=g) + 1.0).double() * 2.0 ** e).float()
    ts, rest = terms(x * 2.0 ** 24)
    assert not rest.any()
    tiny = 2.0 ** -126
    assert all(((t == 0) | (t.abs() >= tiny)).all() for t in ts)
