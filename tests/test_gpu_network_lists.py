"""Chains of propagating layers through cb_network_forward, whose product kernels extract the next stage's index list on the
side, against the same layers called one by one: outputs, maps, lists and counts are the same bits."""
import numpy as np
import pytest
import torch

import synth_inputs as syn

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1808_05488_amd as cb
    from parity import to_dev

# stages: (output channels, filter size, stride, padding, pooling window or 0, pixel-major copy kept)
CHAINS = {
    "pooled": (3, 91, 133, [(32, 3, 1, 1, 2, True), (64, 3, 1, 1, 0, True), (64, 3, 1, 1, 2, True), (40, 3, 1, 1, 0, False)]),
    "wide rows and several workgroups": (4, 300, 519, [(16, 7, 1, 3, 2, True), (32, 5, 1, 2, 0, True), (16, 3, 1, 1, 0, False)]),
    "many workgroups": (2, 700, 1100, [(16, 3, 1, 1, 0, True), (16, 3, 1, 1, 2, True), (16, 1, 1, 0, 0, False)]),
    "strides, padding, one column of words": (3, 64, 40, [(32, 3, 1, 1, 0, True), (32, 3, 2, 0, 0, True), (32, 4, 3, 3, 0, False)]),
    "1x1 takes the list over": (3, 45, 70, [(64, 3, 1, 1, 0, True), (64, 1, 1, 0, 0, True), (32, 3, 1, 1, 2, True), (8, 1, 1, 0, 0, False)]),
    "window of three": (3, 60, 75, [(32, 3, 1, 1, 3, True), (32, 3, 1, 1, 0, False)]),
    "channel-first products": (3, 60, 75, [(24, 3, 1, 1, 2, False), (20, 3, 1, 1, 0, False), (16, 3, 1, 1, 0, False)]),
    "a filter taller than a workgroup's part of the map": (2, 300, 4500, [(16, 1, 1, 0, 0, True), (8, 31, 1, 15, 0, False)]),
}


def _build(chain, bf16):
    c, h, w, stages = chain
    rng = np.random.default_rng(c + h)
    layers, pools = [], []
    for i, (o, k, s, p, win, keep) in enumerate(stages):
        wt = (rng.standard_normal((o, c, k, k)) * np.sqrt(2.0 / (c * k * k))).astype(np.float32)
        b = (rng.standard_normal(o) * 0.1).astype(np.float32)
        prev = i > 0 and stages[i - 1][5]
        both = keep and o >= (32 if bf16 else 16) and i + 1 < len(stages)
        gather = bool(prev and c >= (32 if bf16 else 16) and k * k <= 60)
        layers.append(cb.Layer(to_dev(wt, bf16), to_dev(b, bf16), s, p, h, w, True, mode=cb.CB_PROPAGATE if i else cb.CB_CLOSED_LOOP,
                               keep_output_channel_last=both, gather_channel_last=gather))
        pools.append(cb.Pool(layers[-1], win) if win else None)
        c, h, w = o, layers[-1].Ho, layers[-1].Wo
        if win:
            h, w = -(-h // win), -(-w // win)
    return layers, pools


def _one_by_one(layers, pools, x, tau):
    out = None
    for i, (L, p) in enumerate(zip(layers, pools)):
        out = L.process_frame(x, tau) if i == 0 else L.process_frame_propagated(x, pools[i - 1] or layers[i - 1])
        x = out if p is None else p.process()
    return x


@pytest.mark.parametrize("spins", [1 << 20, 0])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("name", list(CHAINS))
def test_chain_against_single_calls(name, bf16, spins):
    print("network lists:", name, bf16, spins, flush=True)
    chain = CHAINS[name]
    c, h, w, stages = chain
    tau = 0.02
    _, frames = syn.random_layer_case(h, c, 1, 1, 1, 0, h, w, 6, change_prob=0.004, noise_std=0.003)
    frames = [to_dev(f, bf16) for f in frames]
    la, pa = _build(chain, bf16)
    lb, pb = _build(chain, bf16)
    net = cb.Network(la, pa)
    cb.cb_set_scan_wait_limit(spins)
    try:
        for t, f in enumerate(frames):
            if t == 3:                               # a frame that only the first layer sees: the others recompute everything next
                la[0].process_frame(f, tau)
                lb[0].process_frame(f, tau)
                continue
            if t == 4 and len(la) > 2:
                la[1].reset()
                lb[1].reset()
            got = net.forward(f, [tau] * len(la))
            ref = _one_by_one(lb, pb, f, tau)
            assert torch.equal(got, ref), (name, t)
            for i, (a, b) in enumerate(zip(la, lb)):
                for u, v in zip(a.changes_host(), b.changes_host()):
                    assert np.array_equal(u, v), (name, t, i)
                if pa[i] is not None:
                    assert torch.equal(pa[i].changes(), pb[i].changes()), (name, t, i)
    finally:
        cb.cb_set_scan_wait_limit(1 << 20)
    if spins == 0 and name == "many workgroups":
        assert sum(L.stats()["scan_recounts"] for L in la) > 0


def test_captured_network_frames_replay():
    """Two frames per capture; every replay against the same frames called one by one."""
    chain = CHAINS["pooled"]
    c, h, w, _ = chain
    _, frames = syn.random_layer_case(5, c, 1, 1, 1, 0, h, w, 9, change_prob=0.01, noise_std=0.003)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        frames = [to_dev(f, False) for f in frames]
        la, pa = _build(chain, False)
        lb, pb = _build(chain, False)
        net = cb.Network(la, pa)
        taus = [0.02] * len(la)
        for f in frames[:2]:
            net.forward(f, taus)
            _one_by_one(lb, pb, f, 0.02)
        bufs = [torch.empty_like(frames[0]) for _ in range(2)]
        res = [torch.empty_like(net.forward(frames[1], taus)) for _ in range(2)]
        _one_by_one(lb, pb, frames[1], 0.02)
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            for i in range(2):
                res[i].copy_(net.forward(bufs[i], taus))
        for t in range(2, 8, 2):
            for i in range(2):
                bufs[i].copy_(frames[t + i])
            g.replay()
            st.synchronize()
            for i in range(2):
                assert torch.equal(res[i], _one_by_one(lb, pb, frames[t + i], 0.02)), (t, i)
                st.synchronize()
