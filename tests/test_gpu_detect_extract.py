"""The index list extracted inside the launch of change detection, against the oracle: maps whose last word and last group of 16
pixels are partly filled, rows that no output reads, paddings beyond the filter, one workgroup and many; and frames of which some take the launches
one by one (a wait limit of 0), some are timed, some detect at listed pixels, some are full updates."""
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


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("widths", [(3, 5, 4), (16, 32, 20), (24, 64, 8), (8, 100, 6), (4, 128, 6), (6, 200, 5), (3, 256, 4), (5, 300, 3), (3, 512, 3)])
def test_chained_layers(widths, bf16):
    """Detection at the producer's listed pixels, directly and through a pooling stage, against detection of everything in layers of their own;
    frames without a change, frames that take the launches one by one, and a frame in which everything changes."""
    c, mid, o = widths
    print("chained", widths, bf16, flush=True)
    H, W = 61, 93
    rng = np.random.default_rng(mid)
    mk = lambda n, m, k: to_dev((rng.standard_normal((n, m, k, k)) * np.sqrt(2.0 / (m * k * k))).astype(np.float32), bf16)
    w0, w1, w2 = mk(mid, c, 3), mk(o, mid, 3), mk(o, mid, 5)
    first = cb.Layer(w0, None, 1, 1, H, W, True)
    pool = cb.Pool(first, 2)
    direct = [cb.Layer(w1, None, 2, 1, H, W, True) for _ in range(2)]
    pooled = [cb.Layer(w2, None, 1, 2, pool.Hp, pool.Wp, False) for _ in range(2)]
    _, frames = syn.random_layer_case(mid, c, 1, 1, 1, 0, H, W, 9, change_prob=0.02, noise_std=0.003)
    frames[3] = frames[2]
    frames[6] = frames[5] + 1.0
    try:
        for t, f in enumerate(frames):
            x = first.process_frame(to_dev(f, bf16), 0.02)
            y = pool.process()
            cb.cb_set_scan_wait_limit(0 if t in (4, 7) else 1 << 20)      # one by one
            for L in (direct[0], pooled[0]):
                cb.cb_layer_set_timing(L.handle, t in (5, 7))
            direct[0].process_frame_chained(x, first, 0.02)
            pooled[0].process_frame_chained(y, pool, 0.02)
            cb.cb_set_scan_wait_limit(1 << 20)
            direct[1].process_frame(x, 0.02)
            pooled[1].process_frame(y, 0.02)
            for a, b in (direct, pooled):
                for u, v in zip(a.changes_host(), b.changes_host()):
                    assert np.array_equal(u, v), (widths, t)
                assert a.stats()["n_changed_in"] == b.stats()["n_changed_in"], (widths, t)
                assert torch.equal(a.state(), b.state()), (widths, t)
                (so, oo), (sr, orf) = a.export_state(), b.export_state()
                assert torch.equal(oo, orf), (widths, t)
    finally:
        cb.cb_set_scan_wait_limit(1 << 20)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("geom", GEOMS)
def test_blocks_taken_by_workgroups_that_wait(geom, bf16):
    """With a wait limit of one poll the workgroups that extract are numbered first and detect themselves what no other has begun: the same maps, lists,
    states and outputs."""
    C, O, k, s, pad, H, W = geom
    print("taken blocks", geom, bf16, flush=True)
    spec, frames = syn.random_layer_case(C + H, C, O, k, s, pad, H, W, 5, change_prob=0.03)
    p = Pair(spec, H, W, bf16=bf16)
    q = Pair(spec, H, W, bf16=bf16, feed_forward=True)
    try:
        for t, f in enumerate(frames):
            cb.cb_set_scan_wait_limit(1 if t != 3 else 1 << 20)
            p.step(f, 0.02, tag=f"{geom} frame {t}")
            q.step(f, 0.02, tag=f"feed-forward {geom} frame {t}")
    finally:
        cb.cb_set_scan_wait_limit(1 << 20)
    if (C, H) == (33, 400) and not bf16:                        # (four times the workgroups that begin at once)
        assert p.g.stats()["scan_recounts"] > 0


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("widths", [(3, 5, 4), (16, 32, 20), (8, 100, 6), (4, 128, 6), (6, 200, 5), (3, 256, 4), (5, 300, 3)])
def test_listed_blocks_taken_by_workgroups_that_wait(widths, bf16):
    """Detection at listed pixels likewise, directly and through a pooling stage, against detection of everything."""
    c, mid, o = widths
    print("taken listed blocks", widths, bf16, flush=True)
    H, W = 301, 403
    rng = np.random.default_rng(mid)
    mk = lambda n, m, k: to_dev((rng.standard_normal((n, m, k, k)) * np.sqrt(2.0 / (m * k * k))).astype(np.float32), bf16)
    w0, w1, w2 = mk(mid, c, 3), mk(o, mid, 3), mk(o, mid, 5)
    first = cb.Layer(w0, None, 1, 1, H, W, True)
    pool = cb.Pool(first, 2)
    direct = [cb.Layer(w1, None, 2, 1, H, W, True) for _ in range(2)]
    pooled = [cb.Layer(w2, None, 1, 2, pool.Hp, pool.Wp, False) for _ in range(2)]
    _, frames = syn.random_layer_case(mid, c, 1, 1, 1, 0, H, W, 7, change_prob=0.02, noise_std=0.003)
    frames[2] = frames[1]
    frames[4] = frames[3] + 1.0
    try:
        for t, f in enumerate(frames):
            cb.cb_set_scan_wait_limit(1 << 20)
            x = first.process_frame(to_dev(f, bf16), 0.02)
            y = pool.process()
            direct[1].process_frame(x, 0.02)
            pooled[1].process_frame(y, 0.02)
            cb.cb_set_scan_wait_limit(1 if t != 5 else 1 << 20)
            direct[0].process_frame_chained(x, first, 0.02)
            pooled[0].process_frame_chained(y, pool, 0.02)
            for a, b in (direct, pooled):
                for u, v in zip(a.changes_host(), b.changes_host()):
                    assert np.array_equal(u, v), (widths, t)
                assert a.stats()["n_changed_in"] == b.stats()["n_changed_in"], (widths, t)
                assert torch.equal(a.state(), b.state()), (widths, t)
                assert torch.equal(a.export_state()[1], b.export_state()[1]), (widths, t)
    finally:
        cb.cb_set_scan_wait_limit(1 << 20)
    if mid >= 200:                                              # (more workgroups than begin at once)
        assert direct[0].stats()["scan_recounts"] > 0


@pytest.mark.parametrize("limit", [1, 1 << 20])
def test_layers_on_several_streams_at_once(limit):
    """Frames of four layers on streams of their own, nothing waiting between them, against the same layers one after the other."""
    C, H, W = 33, 300, 400
    rng = np.random.default_rng(8)
    w = to_dev((rng.standard_normal((4, C, 3, 3)) / 17).astype(np.float32), False)
    streams = [torch.cuda.Stream() for _ in range(4)]
    cases = [[to_dev(f, False) for f in syn.random_layer_case(20 + i, C, 4, 3, 1, 1, H, W, 6, change_prob=0.02)[1]] for i in range(4)]
    torch.cuda.synchronize()

    def build():
        layers = []
        for s in streams:
            with torch.cuda.stream(s):
                layers.append(cb.Layer(w, None, 1, 1, H, W, True))
        return layers

    a, b = build(), build()
    cb.cb_set_scan_wait_limit(limit)
    try:
        for t in range(6):
            for i in range(4):
                with torch.cuda.stream(streams[i]):
                    a[i].process_frame(cases[i][t], 0.02)
        torch.cuda.synchronize()
    finally:
        cb.cb_set_scan_wait_limit(1 << 20)
    for i in range(4):
        with torch.cuda.stream(streams[i]):
            for f in cases[i]:
                out = b[i].process_frame(f, 0.02)
            torch.cuda.synchronize()
            for u, v in zip(a[i].changes_host(), b[i].changes_host()):
                assert np.array_equal(u, v)
            (sa, oa), (sb, ob) = a[i].export_state(), b[i].export_state()
            torch.cuda.synchronize()
            assert torch.equal(sa, sb) and torch.equal(oa, ob)


def test_timed_frames_have_the_launches_of_others():
    """Per-step times are those of the launches that a frame has without them: the list is part of detection, or of the product of the stage before."""
    rng = np.random.default_rng(2)
    w = [to_dev((rng.standard_normal((32, c, 3, 3)) / 12).astype(np.float32), False) for c in (16, 32, 32)]
    layers = [cb.Layer(w[0], None, 1, 1, 120, 160, True, keep_output_channel_last=True), cb.Layer(w[1], None, 1, 1, 120, 160, True),
              cb.Layer(w[2], None, 1, 1, 120, 160, True, mode=cb.CB_PROPAGATE)]
    net = cb.Network(layers, [None] * 3)
    _, frames = syn.random_layer_case(4, 16, 1, 1, 1, 0, 120, 160, 4, change_prob=0.02)
    for L in layers:
        L.set_timing(True)
    for t, f in enumerate(frames):
        net.forward(to_dev(f, False), [0.02] * 3)
        us = [L.stats()["us_step"] for L in layers]
        assert all(u["fused"] > 0 for u in us) and us[0]["detect"] > 0 and us[1]["detect"] > 0
        assert us[0]["dilate"] == us[1]["dilate"] == us[0]["compact"] == us[1]["compact"] == 0, t
        assert (us[2]["dilate"] == 0) == (t > 0), t                # (the first frame is a full update)
    cb.cb_set_scan_wait_limit(0)
    try:
        net.forward(to_dev(frames[0], False), [0.02] * 3)
        assert layers[0].stats()["us_step"]["dilate"] > 0
    finally:
        cb.cb_set_scan_wait_limit(1 << 20)
