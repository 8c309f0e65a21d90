"""Workloads of change-based convolution whose speed is tracked.

Each case is one frame (or one full update) of a layer or of a whole network, called the way a program that plays a
video through the library calls it: the layer, its weights and the device frames exist, the stream has seen a first
frame, and the next frame comes in.  Frames are synthetic (a fixed background, moving textured rectangles with sensor
noise below the threshold, or replaced 16 x 16 blocks) and are played back and forth, so that every pass is a real
transition.

`exact` restates the method in float64 with plain torch: threshold against the input state, convolution of the
updated state, 2x2 ceil-mode max-pooling.
"""
from __future__ import annotations

import math
import random

import torch

import paper_1808_05488_amd as cb

TAU = 0.02
NOISE = 0.003
SPEED = 3            # pixels a rectangle moves per frame
N_FRAMES = 6         # frames of a moving scene (two for replaced blocks)

_DT = {"f32": torch.float32, "bf16": torch.bfloat16}

# (output channels, filter size, ReLU, 2x2 pooling behind it) of the two networks, three input channels
_NETS = {
    "seg": [(16, 7, 1, 1), (64, 7, 1, 1), (256, 7, 1, 0), (64, 1, 1, 0), (8, 1, 0, 0)],
    "vgg": [(64, 3, 1, 0), (64, 3, 1, 1), (128, 3, 1, 0), (128, 3, 1, 1), (256, 3, 1, 0), (256, 3, 1, 0),
            (256, 3, 1, 0), (256, 3, 1, 1), (512, 3, 1, 0), (512, 3, 1, 0)],
}


def _layer(name, c_in, c_out, k, h, w, dtype="f32", stride=1, relu=0, how="frame", scene="rects", share=0.02):
    """how: "frame" = the next frame of a closed-loop layer; "full" = a full update (first frame, scene cut);
    "feed_forward" = the next frame of a layer that compares with the previous input.
    scene / share: what changes between two frames, and the share of the pixels it covers."""
    d = {"name": name, "kind": "layer", "c_in": c_in, "c_out": c_out, "k": k, "stride": stride, "h": h, "w": w,
         "dtype": dtype, "relu": relu, "how": how, "scene": scene, "share": share}
    if name is None:
        del d["name"]
    return d


def _net(name, net, h, w, dtype="f32", how="detect", share=0.03):
    """how: "detect" = every layer evaluates the threshold (where its producer wrote); "propagate" = layers after the
    first take over their producer's change map."""
    d = {"name": name, "kind": "net", "net": net, "h": h, "w": w, "dtype": dtype, "how": how, "share": share}
    if name is None:
        del d["name"]
    return d


def listed():
    return [
        # the smallest layer of the configurations: nothing but launches and latency
        _layer("tiny_3to16_48x64_f32", 3, 16, 3, 48, 64, share=0.02),
        # the headline layer: VGA feature map, a few moving objects
        _layer("vga_64to64_f32", 64, 64, 3, 480, 640, share=0.021),
        # the same kind of layer in bfloat16 on a map with an odd number of pixels
        _layer("odd_64to128_271x435_bf16", 64, 128, 3, 271, 435, dtype="bf16", relu=1, share=0.03),
        # strided layer, channel counts that are no powers of two, an odd map
        _layer("stride2_48to96_241x323_f32", 48, 96, 5, 241, 323, stride=2, relu=1, share=0.05),
        # first layer of a segmentation net on full-HD camera frames
        _layer("camera_3to16_1080p_f32", 3, 16, 7, 1080, 1920, relu=1, share=0.03),
        # the largest layer, state beyond every cache, both element types
        _layer("hd_128to128_f32", 128, 128, 3, 1080, 1920, scene="blocks", share=0.02),
        _layer("hd_128to128_bf16", 128, 128, 3, 1080, 1920, dtype="bf16", scene="blocks", share=0.10),
        # a scene cut (or the first frame of a stream): every output of a deep layer is computed
        _layer("cut_256to256_92x164_f32", 256, 256, 3, 92, 164, relu=1, how="full"),
        # a layer that compares with the previous input instead of the input state
        _layer("ff_64to64_240x320_f32", 64, 64, 3, 240, 320, relu=1, how="feed_forward", share=0.03),
        # a filter of more taps than the fused kernels take: matrix generation, GEMM and update by themselves
        _layer("wide_32to32_9x9_240x320_f32", 32, 32, 9, 240, 320, relu=1, share=0.03),
        # whole networks: scene labelling with detection in every layer, a VGG trunk with propagated change maps
        _net("seg_480x640_f32", "seg", 480, 640),
        _net("vgg_368x656_bf16", "vgg", 368, 656, dtype="bf16", how="propagate", share=0.05),
    ]


def _largest():
    works = [(c["dtype"], work(c)) for c in listed()]
    return (max(w["bytes"] for _, w in works), {dt: max(w["flops"] for d, w in works if d == dt) for dt in _DT})


def draw(rng):
    max_bytes, max_flops = _largest()
    while True:
        dtype = rng.choice(["f32", "f32", "bf16"])
        h = int(round(math.exp(rng.uniform(math.log(40), math.log(1080)))))
        w = int(round(h * rng.uniform(1.0, 1.8)))
        if rng.random() < 0.2:
            net = rng.choice(["seg", "vgg"])
            h, w = min(max(h, 96), 480), min(max(w, 128), 656)
            c = _net(None, net, h, w, dtype, rng.choice(["detect", "propagate"]), round(rng.uniform(0.01, 0.06), 4))
        else:
            c_in = rng.choice([3, 16, 32, 64, 64, 128, 256, rng.randint(5, 160)])
            c_out = rng.choice([8, 16, 32, 64, 64, 128, 256, rng.randint(5, 160)])
            k = rng.choice([1, 3, 3, 3, 3, 5, 7, 9])
            scene = rng.choice(["rects", "blocks"])
            share = round(math.exp(rng.uniform(math.log(0.003), math.log(0.06 if scene == "rects" else 0.4))), 4)
            how = rng.choice(["frame"] * 8 + ["full", "feed_forward"])
            c = _layer(None, c_in, c_out, k, h, w, dtype, 2 if rng.random() < 0.15 else 1, rng.randint(0, 1), how, scene,
                       share)
        wk = work(c)
        if wk["bytes"] <= max_bytes and wk["flops"] <= max_flops[dtype]:
            return c


# ---------------------------------------------------------------- inputs
def _gen(seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) * 7919 + 12345)
    return g


def _rects(h, w, share):
    """Number and side of the moving rectangles that cover `share` of the pixels."""
    n = 4 if h * w >= 20000 else 2
    side = int(round(math.sqrt(share * h * w / n)))
    return n, max(4, min(side, h // 2, w // 2))


def _frames(case, c, seed, dtype):
    h, w = case["h"], case["w"]
    g = _gen(seed)
    py = random.Random(int(seed))
    if case.get("scene", "rects") == "blocks":
        a = torch.rand((c, h, w), generator=g, device="cuda").to(dtype)
        gh, gw = max(1, h // 16), max(1, w // 16)
        n = max(1, min(gh * gw, int(round(case["share"] * h * w / 256))))
        pick = torch.zeros(gh * gw, dtype=torch.bool, device="cuda")
        pick[torch.randperm(gh * gw, generator=g, device="cuda")[:n]] = True
        m = torch.zeros((h, w), dtype=torch.bool, device="cuda")
        big = pick.view(gh, gw).repeat_interleave(16, 0).repeat_interleave(16, 1)[:h, :w]
        m[:big.shape[0], :big.shape[1]] = big
        fresh = torch.rand((c, h, w), generator=g, device="cuda").to(dtype)
        return [a, torch.where(m, fresh, a).contiguous()]
    n, side = _rects(h, w, case["share"])
    bg = torch.rand((c, h, w), generator=g, device="cuda")
    objs = []
    for i in range(n):
        vy, vx = [(0, SPEED), (SPEED, 0), (0, -SPEED), (-SPEED, 0)][i % 4]
        objs.append([py.randint(0, h - side), py.randint(0, w - side), vy, vx,
                     torch.rand((c, side, side), generator=g, device="cuda")])
    frames = []
    for _ in range(N_FRAMES):
        f = bg.clone()
        for y, x, _vy, _vx, tex in objs:
            f[:, y:y + side, x:x + side] = tex
        f += torch.randn((c, h, w), generator=g, device="cuda") * NOISE
        frames.append(f.to(dtype).contiguous())
        for o in objs:
            for d, size in ((0, h), (1, w)):
                p = o[d] + o[d + 2]
                if p < 0 or p + side > size:         # bounce
                    o[d + 2] = -o[d + 2]
                    p = min(max(o[d] + o[d + 2], 0), size - side)
                o[d] = p
    return frames


def _weights(shapes, seed, dtype):
    g = _gen(seed + 500000)
    out = []
    for o, c, k in shapes:
        wt = torch.randn((o, c, k, k), generator=g, device="cuda") * math.sqrt(2.0 / (c * k * k))
        out.append((wt.to(dtype).contiguous(), (torch.randn((o,), generator=g, device="cuda") * 0.1).to(dtype)))
    return out


def _net_layers(net):
    c, out = 3, []
    for o, k, relu, pool in _NETS[net]:
        out.append((c, o, k, relu, pool))
        c = o
    return out


# ---------------------------------------------------------------- one pass
class _State:
    """What the playing program holds: the frames, where it is, and the layer or network."""

    def __init__(self, case, frames):
        self.case, self.frames, self.t = case, frames, 0

    def next_frame(self):
        self.t += 1
        n = len(self.frames)
        k = self.t % (2 * n - 2)
        return self.frames[k if k < n else 2 * n - 2 - k]


def prepare(case, seed):
    dt = _DT[case["dtype"]]
    if case["kind"] == "layer":
        s = _State(case, _frames(case, case["c_in"], seed, dt))
        (wt, b), = _weights([(case["c_out"], case["c_in"], case["k"])], seed, dt)
        mode = cb.CB_FEED_FORWARD if case["how"] == "feed_forward" else cb.CB_CLOSED_LOOP
        s.layer = cb.Layer(wt, b, case["stride"], case["k"] // 2, case["h"], case["w"], bool(case["relu"]), mode=mode)
        s.layer.process_frame(s.frames[0], TAU)
        return s
    s = _State(case, _frames(case, 3, seed, dt))
    spec = _net_layers(case["net"])
    ws = _weights([(o, c, k) for c, o, k, _, _ in spec], seed, dt)
    propagate = case["how"] == "propagate"

    def both_ways(ch):                               # whose output can also be kept pixel by pixel
        return propagate and ch >= (16 if case["dtype"] == "f32" else 32) and ch & (ch - 1) == 0

    h, w, layers, pools = case["h"], case["w"], [], []
    for i, ((c, o, k, relu, pool), (wt, b)) in enumerate(zip(spec, ws)):
        layers.append(cb.Layer(wt, b, 1, k // 2, h, w, bool(relu),
                               mode=cb.CB_PROPAGATE if propagate and i else cb.CB_CLOSED_LOOP,
                               keep_output_channel_last=both_ways(o) and i + 1 < len(spec),
                               gather_channel_last=bool(i) and both_ways(c)))
        pools.append(cb.Pool(layers[-1], 2) if pool else None)
        if pool:
            h, w = (h + 1) // 2, (w + 1) // 2
    s.net = cb.Network(layers, pools)
    s.taus = [TAU] * len(layers)
    s.net.forward(s.frames[0], s.taus)
    return s


def run(s):
    x = s.next_frame()
    if s.case["kind"] == "net":
        return {"out": s.net.forward(x, s.taus)}
    if s.case["how"] == "full":
        s.layer.reset()
    out = s.layer.process_frame(x, TAU)
    return {"out": out, "state": s.layer.state()}


# ---------------------------------------------------------------- what a pass cannot do without
def _changed(case, h, w):
    """Boxes (height, width, count) that change between two frames."""
    if case.get("scene", "rects") == "blocks":
        n = max(1, min(max(1, h // 16) * max(1, w // 16), int(round(case["share"] * h * w / 256))))
        return (16.0, 16.0, n)
    n, side = _rects(h, w, case["share"])
    return (side + SPEED / 2, side + SPEED / 2, n)


def work(case):
    b = 4 if case["dtype"] == "f32" else 2
    h, w = case["h"], case["w"]
    bh, bw, n = _changed(case, h, w)
    if case["kind"] == "layer":
        c, o, k, s = case["c_in"], case["c_out"], case["k"], case["stride"]
        p = h * w
        ho, wo = (h + 2 * (k // 2) - k) // s + 1, (w + 2 * (k // 2) - k) // s + 1
        m = min(float(p), bh * bw * n)
        no = min(float(ho * wo), (bh + k - 1) * (bw + k - 1) / (s * s) * n)
        if case["scene"] == "blocks":                # neighbouring blocks share their borders
            no = ho * wo * (1.0 - math.exp(-no / (ho * wo)))
        if case["how"] == "full":
            m, no = p, ho * wo
        read = c * p * b * (1 if case["how"] == "full" else 2)
        wrote = c * b * (p if case["how"] == "feed_forward" else m)
        return {"bytes": read + wrote + o * no * b + o * c * k * k * b, "flops": 2.0 * o * c * k * k * no}
    total, flops = 2.0 * 3 * h * w * b, 0.0          # the frame and the first layer's state
    for i, (c, o, k, _relu, pool) in enumerate(_net_layers(case["net"])):
        m = min(float(h * w), bh * bw * n)
        bh, bw = bh + k - 1, bw + k - 1
        no = min(float(h * w), bh * bw * n)
        if i:
            total += c * m * b * (3 if case["how"] == "detect" else 1)    # input, state, state update
        total += o * no * b + o * c * k * k * b
        flops += 2.0 * o * c * k * k * no
        if pool:
            total += o * no * b * 1.25
            h, w, bh, bw = (h + 1) // 2, (w + 1) // 2, bh / 2 + 1, bw / 2 + 1
    return {"bytes": total, "flops": flops}


def tolerance(case):
    # (two back ends of the library against each other, 42 cases: single layers differ by up to 1.9e-6, largest
    # difference 1.5e-5, in float32 and 8e-5 / 7.8e-3, one step of the type, in bfloat16; networks 1.3e-6 and 4.1e-3 / 0.03)
    if case["kind"] == "net":
        # a threshold decision may fall differently for a value within rounding of it, and the layers behind follow
        return {"rel": 1e-4, "max": 0.1} if case["dtype"] == "f32" else {"rel": 1.6e-2, "max": 0.2}
    # sums of up to a few thousand products in float32; one rounding to bfloat16 of a sum that may lie on a tie
    return {"rel": 1e-5, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 5e-4, "max": 2e-2}


# ---------------------------------------------------------------- the method in float64
def _conv64(x, wt, bias, stride, pad, relu):
    o, c, k, _ = wt.shape
    ho, wo = (x.shape[1] + 2 * pad - k) // stride + 1, (x.shape[2] + 2 * pad - k) // stride + 1
    xp = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    y = bias.double().view(o, 1).repeat(1, ho * wo)
    wd = wt.double()
    for j in range(k):
        for i in range(k):
            tap = xp[:, j:j + (ho - 1) * stride + 1:stride, i:i + (wo - 1) * stride + 1:stride].double()
            y.addmm_(wd[:, :, j, i].contiguous(), tap.reshape(c, ho * wo))
            del tap
    return (y.clamp_(min=0) if relu else y).view(o, ho, wo)


def _fires(x, state):
    """Pixels where some channel differs by more than the threshold (compared in float32)."""
    hit = torch.zeros(x.shape[1:], dtype=torch.bool, device=x.device)
    for c in range(x.shape[0]):
        hit |= (x[c].float() - state[c].float()).abs() > torch.tensor(TAU, dtype=torch.float32, device=x.device)
    return hit


def _dilate(hit, k, stride, pad):
    m = torch.nn.functional.max_pool2d(torch.nn.functional.pad(hit.float()[None], (pad, pad, pad, pad)), k, stride)
    return m[0] > 0


def _pool(x):
    return torch.nn.functional.max_pool2d(x[None], 2, 2, ceil_mode=True)[0]


def exact(case, seed):
    dt = _DT[case["dtype"]]
    if case["kind"] == "layer":
        frames = _frames(case, case["c_in"], seed, dt)[:2]
        (wt, b), = _weights([(case["c_out"], case["c_in"], case["k"])], seed, dt)
        k, s, relu = case["k"], case["stride"], case["relu"]
        hit = _fires(frames[1], frames[0])
        if case["how"] == "frame":
            st = torch.where(hit, frames[1], frames[0])
            out = _conv64(st, wt, b, s, k // 2, relu)
        else:
            st = frames[1]
            out = _conv64(st, wt, b, s, k // 2, relu)
            if case["how"] == "feed_forward":
                out = torch.where(_dilate(hit, k, s, k // 2), out, _conv64(frames[0], wt, b, s, k // 2, relu))
        return {"out": out, "state": st}
    frames = _frames(case, 3, seed, dt)[:2]
    spec = _net_layers(case["net"])
    ws = _weights([(o, c, k) for c, o, k, _, _ in spec], seed, dt)
    # what a layer hands on is its cached output, in the element type; the last one's is returned as summed
    x0, x1 = frames
    for i, ((c, o, k, relu, pool), (wt, b)) in enumerate(zip(spec, ws)):
        last = i + 1 == len(spec)
        if i == 0 or case["how"] == "detect":
            st = torch.where(_fires(x1, x0), x1, x0)
        else:
            st = x1
        y1 = _conv64(st, wt, b, 1, k // 2, relu)
        if last:
            return {"out": _pool(y1) if pool else y1}
        y0 = _conv64(x0, wt, b, 1, k // 2, relu)
        x0, x1 = (_pool(y.to(dt).float()).to(dt) if pool else y.to(dt) for y in (y0, y1))
        del y0, y1
