"""Layers whose packed filter matrix is beyond 2 MB: the row tiles are divided among two, four or eight groups of XCDs, according to the listed
pixels, with row and column tiles that do not come out even."""
import pytest
import torch

import synth_inputs as syn

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from parity import Pair


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("geom", [(256, 300, 3, 19, 23), (512, 260, 3, 13, 17), (128, 330, 5, 40, 45), (64, 520, 7, 30, 33), (1024, 1030, 1, 24, 31),
                                  (512, 520, 3, 5, 7), (64, 140, 9, 60, 100)])
@pytest.mark.parametrize("prob", [0.002, 0.1])
def test_row_tiles_divided_among_the_xcds(geom, prob, bf16):
    C, O, k, H, W = geom
    print("long filters", geom, prob, bf16, flush=True)
    spec, frames = syn.random_layer_case(C + O, C, O, k, 1, k // 2, H, W, 3, change_prob=prob)
    p = Pair(spec, H, W, bf16=bf16)
    for t, f in enumerate(frames):
        p.step(f, 0.02, tag=f"{geom} frame {t}")
