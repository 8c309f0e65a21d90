"""The index list extracted inside the launch of change detection, against the oracle: maps whose last word and last group of 16
pixels are partly filled, rows that no output reads, paddings beyond the filter, one workgroup and many; and frames of which some take the launches
one by one (per-step times on, another wait limit), some detect at listed pixels, some are full updates."""
import numpy as np
import pytest
import torch

import synth_inputs as syn

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1808_05488_amd as cb
    from oracle import cb_oracle as orc
    from parity import Pair, to_dev, to_host

# (input channels, output channels, filter size, stride, padding, height, width)
GEOMS = [
    (3, 4, 3, 1, 1, 1, 1), (3, 4, 3, 1, 1, 7, 9), (1, 2, 1, 1, 0, 64, 64), (3, 4, 3, 1, 1, 65, 63), (2, 3, 5, 1, 4, 33, 200),
    (3, 5, 1, 2, 0, 41, 130), (3, 5, 2, 2, 0, 131, 129), (4, 6, 3, 2, 1, 90, 411), (20, 6, 3, 2, 2, 300, 331), (64, 8, 3, 2, 0, 37, 29),
    (70, 6, 3, 1, 1, 10, 10), (100, 6, 3, 1, 1, 9, 113), (128, 6, 1, 1, 0, 63, 130), (200, 6, 3, 1, 1, 5, 13), (300, 6, 3, 1, 2, 21, 23), (512, 4, 3, 2, 1, 46, 82),
    (17, 4, 7, 1, 3, 200, 333), (33, 4, 3, 1, 1, 400, 640), (3, 4, 31, 1, 15, 120, 1000), (2, 3, 3, 1, 1, 1300, 2000), (3, 3, 3, 1, 1, 2, 5000), (3, 3, 3, 1, 1, 5000, 2),
    (140, 3, 3, 1, 1, 240, 300), (600, 3, 1, 1, 0, 20, 30), (3, 4, 3, 3, 1, 50, 60),
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("geom", GEOMS)
def test_list_from_the_launch_of_detection(geom, bf16):
    C, O, k, s, pad, H, W = geom
    print("detect and extract", geom, bf16, flush=True)
    spec, frames = syn.random_layer_case(C + H, C, O, k, s, pad, H, W, 5, change_prob=0.03)
    p = Pair(spec, H, W, bf16=bf16)
    for t, f in enumerate(frames):
        p.step(f, 0.02, tag=f"{geom} frame {t}")


def test_launches_together_and_one_by_one():
    C, O, k, s, pad, H, W = 16, 12, 3, 1, 1, 150, 200
    spec, frames = syn.random_layer_case(3, C, O, k, s, pad, H, W, 16, change_prob=0.02)
    p = Pair(spec, H, W)
    rng = np.random.default_rng(1)
    try:
        for t, f in enumerate(frames):
            how = int(rng.integers(0, 4))
            cb.cb_layer_set_timing(p.g.handle, how == 1)
            cb.cb_set_scan_wait_limit(0 if how == 2 else 1 << 20)
            if how == 3:
                p.g.reset()
                p.o.reset()
            p.step(f, 0.02, tag=f"frame {t} how {how}")
    finally:
        cb.cb_set_scan_wait_limit(1 << 20)


def test_many_frames_of_a_vga_layer():
    """Two hundred frames with scattered changes: the list against the map that the same frame detected."""
    C, H, W = 64, 480, 640
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    L = cb.Layer(torch.zeros((1, C, 3, 3), device="cuda"), None, 1, 1, H, W, False)
    x = torch.rand((C, H, W), generator=g, device="cuda")
    for t in range(200):
        L.process_frame(x, 0.02)
        m, mt, idx, n = L.changes_host()
        if t:
            assert np.array_equal(m, hit.cpu().numpy())
        ref = torch.nn.functional.max_pool2d(torch.from_numpy(m).float()[None], 3, 1, 1)[0].numpy() > 0
        assert np.array_equal(mt > 0, ref) and np.array_equal(idx, np.flatnonzero(ref)) and n == idx.size, t
        hit = torch.rand((H, W), generator=g, device="cuda") < 0.01
        hit[40 + t:90 + t, 100:160] = True
        x = torch.where(hit, torch.rand((C, H, W), generator=g, device="cuda") + 2.0 * (t + 1), x)
