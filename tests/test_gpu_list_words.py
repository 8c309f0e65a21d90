"""The words of the dilated map that the extraction beside detection makes, each by one, two or four lanes (csrc/cb_extract.h, fires_shared): filters of 1 to
31 rows and columns, paddings up to 31, widths around whole and half words, both strides, few and many words a workgroup; and the bits that detection at
listed pixels sets, for candidates in one word, in as many as are combined, and in more."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1808_05488_amd as cb

# (filter rows, columns, padding, stride, height, width)
GEOMS = [
    (1, 1, 0, 1, 40, 64), (1, 31, 31, 1, 40, 65), (31, 1, 31, 1, 33, 63), (2, 2, 1, 1, 70, 33), (3, 3, 1, 1, 48, 64), (4, 3, 2, 1, 90, 95), (5, 5, 2, 1, 61, 96),
    (8, 7, 4, 1, 57, 129), (9, 16, 8, 1, 120, 161), (17, 17, 8, 1, 100, 127), (31, 31, 31, 1, 64, 191), (31, 31, 0, 1, 64, 190), (3, 3, 1, 2, 61, 64), (1, 2, 0, 2, 80, 129),
    (7, 5, 3, 2, 99, 255), (31, 31, 31, 2, 70, 333), (9, 9, 4, 1, 240, 320), (3, 3, 1, 1, 700, 1100), (7, 7, 3, 2, 720, 1280), (5, 5, 2, 1, 3, 3000), (3, 3, 31, 1, 1, 1),
]


@pytest.mark.parametrize("geom", GEOMS)
def test_dilated_words_and_list(geom):
    kh, kw, pad, s, H, W = geom
    print("words", geom, flush=True)
    rng = np.random.default_rng(kh * 100 + W)
    L = cb.Layer(torch.ones((1, 1, kh, kw), device="cuda"), None, s, pad, H, W, False)
    x = torch.zeros((1, H, W), device="cuda")
    L.process_frame(x, 0.5)
    for share in (0.0005, 0.02, 0.5):
        hit = rng.random((H, W)) < share
        hit[0, 0] = hit[H - 1, W - 1] = True
        x = x + torch.from_numpy(hit.astype(np.float32))[None].cuda()
        L.process_frame(x, 0.5)
        m, mt, idx, n = L.changes_host()
        assert np.array_equal(m > 0, hit)
        p = torch.nn.functional.pad(torch.from_numpy(hit.astype(np.float32))[None], (pad, pad, pad, pad))
        ref = torch.nn.functional.max_pool2d(p, (kh, kw), s)[0].numpy() > 0
        assert np.array_equal(mt > 0, ref)
        assert n == ref.sum() and np.array_equal(idx, np.flatnonzero(ref))


@pytest.mark.parametrize("W", [1, 2, 61, 62, 63, 64, 65, 66, 67])
@pytest.mark.parametrize("k", [1, 3])
def test_strided_maps_of_half_a_word(k, W):
    """Stride 2, outputs around 32 a row: rows of one half of a word, and of a half and a little more."""
    test_dilated_words_and_list((k, k, k // 2, 2, 29, W))


@pytest.mark.parametrize("channels", [16, 64, 128, 256, 512, 24, 300])
@pytest.mark.parametrize("apart", [1, 3, 5, 33, 97])
def test_bits_of_listed_pixels(channels, apart):
    """Candidates `apart` pixels from each other: all of a wavefront's in one word of 32 pixels, in some, in one each; every second of them fires."""
    H, W = 43, 97
    print("listed bits", channels, apart, flush=True)
    first = cb.Layer(torch.ones((channels, 1, 1, 1), device="cuda"), None, 1, 0, H, W, False)
    eye = torch.zeros((1, channels, 1, 1), device="cuda")
    eye[0, 0] = 1
    layers = [cb.Layer(eye, None, 1, 0, H, W, False) for _ in range(2)]
    x = torch.zeros((1, H, W), device="cuda")
    for t in range(4):
        if t:
            d = torch.zeros(H * W, device="cuda")
            d[t::apart] = 0.2
            d[t::2 * apart] = 1.0
            x = x + d.view(1, H, W)
        y = first.process_frame(x, 0.1)
        layers[0].process_frame_chained(y, first, 0.5)
        layers[1].process_frame(y, 0.5)
        for u, v in zip(layers[0].changes_host(), layers[1].changes_host()):
            assert np.array_equal(u, v), (channels, apart, t)
        assert layers[0].stats()["n_changed_in"] == layers[1].stats()["n_changed_in"]
        assert torch.equal(layers[0].state(), layers[1].state())
