"""Closed-loop layers of any channel count and filter size on the channel-last kernel (CB_BACKEND_AUTO): pixels of the shadow
padded to whole 16-byte pieces, taps that begin anywhere in a stage, filters of more taps than CB_BACKEND_FUSED takes."""
import numpy as np
import pytest
import torch

import synth_inputs as syn

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1808_05488_amd as cb
    from paper_1808_05488_amd.binding import _raw_to_host
    from parity import Pair, split_bound, to_dev, to_host

# (input channels, output channels, filter size, stride, height, width)
GEOMS = [
    (5, 13, 3, 1, 31, 37), (7, 20, 5, 2, 45, 41), (8, 9, 1, 1, 23, 70),            # two pieces a pixel: one group of lanes
    (9, 70, 3, 1, 27, 29), (11, 130, 9, 1, 20, 21), (12, 40, 3, 2, 33, 66),
    (16, 33, 3, 1, 40, 44), (17, 45, 3, 1, 67, 73), (24, 24, 9, 1, 60, 50), (31, 12, 3, 1, 130, 140),
    (33, 64, 3, 1, 90, 97), (48, 96, 5, 2, 51, 63), (63, 72, 3, 1, 75, 81), (65, 17, 3, 1, 18, 20),
    (96, 140, 3, 1, 62, 99), (100, 100, 1, 1, 130, 126), (127, 30, 3, 1, 70, 130), (130, 16, 5, 1, 21, 30),
    (200, 50, 3, 1, 30, 31), (260, 24, 3, 1, 20, 110), (500, 8, 3, 1, 12, 13), (515, 70, 1, 1, 16, 17), (520, 6, 1, 1, 256, 260),
    (3, 16, 9, 1, 61, 67), (32, 32, 9, 1, 50, 60), (16, 5, 31, 1, 40, 42), (2, 6, 11, 3, 50, 51),
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("geom", GEOMS)
def test_any_channel_count(geom, bf16):
    C, O, k, s, H, W = geom
    print("any channels", geom, bf16, flush=True)
    spec, frames = syn.random_layer_case(C + O + k, C, O, k, s, k // 2, H, W, 4, change_prob=0.03, noise_std=0.004)
    p = Pair(spec, H, W, bf16=bf16)
    for t, f in enumerate(frames):
        p.step(f, 0.02, tag=f"{geom} bf16={bf16} frame {t}")


def test_filter_of_one_row():
    rng = np.random.default_rng(4)
    for kh, kw, C in ((1, 31, 20), (31, 1, 12), (5, 16, 24)):
        spec, frames = syn.random_layer_case(kh, C, 12, 3, 1, 2, 40, 45, 3, change_prob=0.03)
        spec.weight = (rng.standard_normal((12, C, kh, kw)) * 0.1).astype(np.float32)
        p = Pair(spec, 40, 45)
        for t, f in enumerate(frames):
            p.step(f, 0.02, tag=f"{kh}x{kw} frame {t}")


def test_state_beyond_the_last_level_cache():
    """The state update as a kernel of its own: 130 channels are one chunk of 128 and a piece with two channels behind the last."""
    spec, frames = syn.random_layer_case(9, 130, 3, 1, 1, 0, 520, 520, 3, change_prob=0.01)
    p = Pair(spec, 520, 520)
    for t, f in enumerate(frames):
        p.step(f, 0.02, tag=f"frame {t}")


def test_import_and_chained_detection():
    """A consumer with 24 channels behind a producer: its shadow is rebuilt from an imported state, then updated at listed pixels."""
    a, frames = syn.random_layer_case(5, 6, 24, 3, 1, 1, 40, 50, 5, change_prob=0.03)
    b, _ = syn.random_layer_case(6, 24, 10, 3, 1, 1, 40, 50, 1)
    la, lb = (cb.Layer(to_dev(s.weight, False), None if s.bias is None else to_dev(s.bias, False), 1, 1, 40, 50, True) for s in (a, b))
    pb = Pair(b, 40, 50)
    for t, f in enumerate(frames):
        mid = la.process_frame(to_dev(f, False), 0.02)
        out = to_host(lb.process_frame_chained(mid, la, 0.01))
        ref, _ = pb.step(to_host(mid), 0.01, tag=f"frame {t}")
        assert np.array_equal(out, ref)
        if t == 1:                                   # moves into a fresh layer
            st, o = lb.export_state()
            lb = cb.Layer(to_dev(b.weight, False), None if b.bias is None else to_dev(b.bias, False), 1, 1, 40, 50, True)
            lb.import_state(st, o)


@pytest.mark.parametrize("C", [5, 24, 100])
def test_special_values_and_accuracy(C):
    rng = np.random.default_rng(C)
    O, H, W = 40, 33, 35
    x = rng.standard_normal((C, H, W)).astype(np.float32)
    w = (rng.standard_normal((O, C, 3, 3)) / 30).astype(np.float32)
    L = cb.Layer(to_dev(w, False), None, 1, 1, H, W, False)
    ref = torch.nn.functional.conv2d(torch.from_numpy(x)[None].double(), torch.from_numpy(w).double(), None, 1, 1)[0].numpy()
    got = to_host(L.process_frame(to_dev(x, False), 0.0)).astype(np.float64)
    assert np.linalg.norm(got - ref) <= split_bound(9 * C) * np.linalg.norm(ref)
    for v in (np.inf, np.nan, np.float32(3e38)):
        y = x.copy()
        y[C - 1, 7, 9] = v
        L.reset()
        got = to_host(L.process_frame(to_dev(y, False), 0.0)).astype(np.float64)
        with np.errstate(all="ignore"):
            ref = torch.nn.functional.conv2d(torch.from_numpy(y)[None].double(), torch.from_numpy(w).double(), None, 1, 1)[0].numpy()
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
        fin = np.isfinite(ref)
        mag = np.abs(ref[fin]) + np.abs(ref[fin]).max()
        assert (np.abs(got[fin] - ref[fin]) <= (9 * C + 1) * 2.0 ** -24 * mag).all()
    L = cb.Layer(to_dev(np.where(np.arange(O)[:, None, None, None] == 3, np.inf, w).astype(np.float32), False), None, 1, 1, H, W, False)
    assert not np.isfinite(to_host(L.process_frame(to_dev(np.abs(x) + 1, False), 0.0))[3]).any()


def test_matrices_on_request():
    """A filter of 81 taps: X' and Y' of the last frame, as the explicit back end has them, also with one column chunk of several."""
    spec, frames = syn.random_layer_case(3, 8, 12, 9, 1, 4, 40, 50, 3, change_prob=0.02)
    for small in (False, True):
        size = cb.cb_layer_min_scratch_bytes(cb.make_desc(8, 12, 9, 9, 1, 4, 40, 50)) if small else None
        assert size is None or size == cb.cb_layer_min_scratch_bytes(cb.make_desc(8, 12, 9, 9, 1, 4, 40, 50, backend=1))
        auto, expl = Pair(spec, 40, 50, scratch_bytes=size), Pair(spec, 40, 50, scratch_bytes=size, backend=1)
        for t, f in enumerate(frames):
            auto.step(f, 0.02, tag=f"frame {t}")
            expl.step(f, 0.02, tag=f"frame {t}")
            got = []
            for p in (auto, expl):
                xp, yp, ldn = cb.cb_layer_matrices(p.g.handle)
                ld, ncols, nsplit = [int(v) for v in _raw_to_host(ldn, 3, p.g.device)]
                got.append(((ld, ncols, nsplit), _raw_to_host(xp, 648 * ld, p.g.device), _raw_to_host(yp, 12 * ld * nsplit, p.g.device)))
            assert got[0][0] == got[1][0]
            assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2])


def test_matrices_behind_a_reset_and_an_import():
    """Behind a reset the matrices of the last frame, as the explicit back end still has them; behind an import, whose change set is empty, none."""
    spec, frames = syn.random_layer_case(3, 8, 12, 9, 1, 4, 40, 50, 3, change_prob=0.02)
    auto, expl = Pair(spec, 40, 50), Pair(spec, 40, 50, backend=1)

    def matrices(p):
        xp, yp, ldn = cb.cb_layer_matrices(p.g.handle)
        ld, ncols, nsplit = [int(v) for v in _raw_to_host(ldn, 3, p.g.device)]
        return (ld, ncols, nsplit), _raw_to_host(xp, 648 * ld, p.g.device), _raw_to_host(yp, 12 * ld * nsplit, p.g.device)

    for t, f in enumerate(frames):
        for p in (auto, expl):
            p.step(f, 0.02, tag=f"frame {t}")
            p.g.reset()
        a, b = matrices(auto), matrices(expl)
        assert a[0] == b[0] and a[0][1] > 0 and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
        for p in (auto, expl):
            p.o.reset()
    auto.g.import_state(auto.g.state().clone(), auto.g_out.clone())
    assert int(_raw_to_host(cb.cb_layer_matrices(auto.g.handle)[2], 3, auto.g.device)[1]) == 0


def test_what_the_fused_back_end_refused_it_refuses():
    for kw in ({"backend": 2}, {"keep_output_channel_last": True}, {"gather_channel_last": True, "mode": cb.CB_PROPAGATE}):
        with pytest.raises(Exception):
            cb.cb_layer_workspace_bytes(cb.make_desc(32, 32, 9, 9, 1, 4, 40, 50, **kw))
