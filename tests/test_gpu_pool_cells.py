"""2 x 2 pooling of a change-based layer against the dense pool of its output: maps of one row, one column and odd sizes, channel counts around the four that an item has, with
and without a pixel-major copy, frames that list everything, something and nothing."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_1808_05488_amd as cb


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 1, 7), (4, 9, 1), (5, 2, 2), (8, 7, 9), (13, 33, 65), (32, 61, 93), (64, 120, 161), (1, 700, 1100), (260, 17, 16)])
def test_pooled_cells(shape, bf16):
    O, H, W = shape
    print("pool", shape, bf16, flush=True)
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(O + H)
    w = torch.randn((O, 2, 1, 1), generator=g, device="cuda").to(dt)
    both = O & (O - 1) == 0 and O >= 32
    for copy in ((False, True) if both else (False,)):
        L = cb.Layer(w, None, 1, 0, H, W, False, keep_output_channel_last=copy)
        P = cb.Pool(L, 2)
        x = torch.rand((2, H, W), generator=g, device="cuda").to(dt)
        for t in range(4):
            y = L.process_frame(x, 0.01)
            out = P.process().clone()
            ref = torch.nn.functional.max_pool2d(y[None].float(), 2, 2, ceil_mode=True)[0]
            assert torch.equal(out.float(), ref), (shape, bf16, copy, t)
            if t < 2:
                hit = torch.rand((H, W), generator=g, device="cuda") < 0.1
                x = torch.where(hit, torch.rand((2, H, W), generator=g, device="cuda").to(dt), x)
