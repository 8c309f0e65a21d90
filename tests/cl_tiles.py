"""Layers whose full update runs each tile of the channel-last fused kernel (csrc/cb_cl_rules.h): instance (rows of its widest
tile), number of the tile, bfloat16, input channels, output channels, filter size, height, width.  Output channels and
listed pixels fill the last row and column tile, and the filters the last stage, only in part.  test_cl_rules.py checks on the host
that each layer picks the tile it stands for and that no tile is missing; test_gpu_parity.py runs them."""
TILE_CASES = [
    (16, 0, False, 16, 13, 3, 7, 9), (16, 1, False, 16, 13, 3, 133, 143), (16, 2, False, 16, 13, 3, 251, 257),
    (32, 0, False, 16, 24, 3, 7, 9), (32, 1, False, 16, 24, 3, 49, 53), (32, 2, False, 16, 24, 3, 91, 99),
    (32, 3, False, 16, 24, 3, 133, 143),
    (64, 0, False, 16, 45, 3, 7, 9), (64, 1, False, 16, 45, 3, 37, 41), (64, 2, False, 16, 45, 3, 67, 73),
    (64, 3, False, 16, 45, 3, 91, 99),
    (128, 0, False, 16, 72, 3, 7, 9), (128, 1, False, 16, 100, 3, 25, 27), (128, 2, False, 32, 72, 3, 49, 53),
    (128, 3, False, 3, 72, 3, 75, 81), (128, 4, False, 32, 72, 3, 91, 99),
    (16, 0, True, 32, 13, 3, 7, 9), (16, 1, True, 32, 13, 3, 67, 73), (16, 2, True, 32, 13, 3, 133, 143),
    (32, 0, True, 32, 24, 3, 7, 9), (32, 1, True, 32, 24, 3, 67, 73), (32, 2, True, 32, 24, 3, 97, 103),
    (32, 3, True, 32, 30, 3, 133, 143),
    (64, 0, True, 32, 45, 3, 7, 9), (64, 1, True, 32, 45, 3, 37, 41), (64, 2, True, 64, 45, 3, 67, 73),
    (64, 3, True, 64, 50, 3, 91, 99),
    (128, 0, True, 32, 72, 3, 7, 9), (128, 1, True, 64, 100, 3, 41, 43), (128, 2, True, 64, 72, 3, 49, 53),
    (128, 3, True, 32, 140, 3, 91, 99), (128, 4, True, 64, 130, 3, 145, 153),
    (129, 5, True, 32, 140, 1, 251, 263), (129, 5, True, 32, 200, 3, 251, 263),
]

# The instance of bfloat16 layers with large maps: a layer (input channels, output channels, filter size, height, width) and the sides of
# square regions whose change lists the pixels for each of its tiles.
LARGE_MAP_LAYER = (64, 130, 3, 251, 263)
LARGE_MAP_REGIONS = [(10, 0), (27, 1), (43, 2), (80, 3), (118, 4), (215, 5)]
