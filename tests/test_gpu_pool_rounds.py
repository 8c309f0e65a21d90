"""2 x 2 pooling: lists whose rounds are made of eight items and of the channels of a tile (csrc/cb_update.hip), and the pixel-major copy, handed on bit for bit by a consumer that gathers from it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1808_05488_amd as cb


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", [(16, 61, 67), (32, 61, 93), (36, 61, 93), (48, 40, 200), (64, 120, 161), (100, 50, 51)])
def test_rounds_and_copies(shape, bf16):
    O, H, W = shape
    print("pool", shape, bf16, flush=True)
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(O + H)
    w = torch.randn((O, 2, 1, 1), generator=g, device="cuda").to(dt)
    both = O & (O - 1) == 0 and O >= (32 if bf16 else 16)
    for copy in ((False, True) if both else (False,)):
        L = cb.Layer(w, None, 1, 0, H, W, False, keep_output_channel_last=copy)
        P = cb.Pool(L, 2)
        reader = None
        if copy:
            reader = cb.Layer(torch.eye(O, device="cuda").to(dt).view(O, O, 1, 1).contiguous(), None, 1, 0, (H + 1) // 2, (W + 1) // 2, False, mode=cb.CB_PROPAGATE,
                              gather_channel_last=True)
        x = torch.rand((2, H, W), generator=g, device="cuda").to(dt)
        for t in range(4):
            y = L.process_frame(x, 0.01)
            pooled = P.process()
            out = pooled.clone()
            ref = torch.nn.functional.max_pool2d(y[None].float(), 2, 2, ceil_mode=True)[0]
            assert torch.equal(out.float(), ref), (shape, bf16, copy, t)
            if reader:
                assert torch.equal(reader.process_frame_propagated(pooled, P), out), (shape, bf16, t)
            if t < 2:
                hit = torch.rand((H, W), generator=g, device="cuda") < 0.1
                x = torch.where(hit, torch.rand((2, H, W), generator=g, device="cuda").to(dt), x)
