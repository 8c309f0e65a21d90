"""The words of the dilated map that the extraction beside detection makes, each by one, two or four lanes (csrc/cb_extract.h, fires_shared): filters of 1 to
31 rows and columns, paddings up to 31, widths around whole and half words, both strides, few and many words a workgroup."""
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
