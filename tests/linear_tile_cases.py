"""Shapes of the linear layer with the tile that the planner has to choose for them: one per tile shape, uncut and cut along k, with
one token tile and with several; ragged in tokens and (where it can be) in features, odd and even numbers of k stages."""

# (tokens, out_features, in_features): (features, tokens of the tile, one token tile covers the batch, pieces of k)
LARGE = {
    (65, 128, 64): (128, 64, False, 1), (300, 384, 704): (128, 64, False, 1), (65, 384, 704): (128, 64, False, 2),
    (1025, 2176, 704): (192, 64, False, 1), (129, 3968, 3008): (192, 64, False, 4), (257, 12416, 704): (256, 64, False, 1),
    (900, 3968, 704): (128, 128, False, 1), (900, 1152, 2496): (128, 128, False, 3), (65, 8320, 1984): (128, 128, True, 3),
    (1025, 3968, 704): (128, 192, False, 1), (1025, 1280, 4032): (128, 192, False, 4), (129, 6272, 3008): (128, 192, True, 4),
    (1025, 6272, 704): (128, 256, False, 1), (1025, 2176, 8128): (128, 256, False, 3), (193, 8320, 3008): (128, 256, True, 3),
    (577, 8320, 704): (192, 128, False, 1), (577, 1920, 8128): (192, 128, False, 5), (65, 8320, 6080): (192, 128, True, 5),
    (900, 8320, 704): (192, 192, False, 1), (1025, 1920, 6080): (192, 192, False, 4), (129, 8320, 8128): (192, 192, True, 5),
    (1000, 12160, 64): (192, 256, False, 1), (450, 6272, 6080): (192, 256, False, 3), (193, 12416, 5056): (192, 256, True, 3),
    (577, 12416, 704): (256, 128, False, 1), (577, 2560, 8128): (256, 128, False, 5), (65, 12416, 4032): (256, 128, True, 5),
    (1025, 8320, 704): (256, 192, False, 1), (577, 4992, 6080): (256, 192, False, 3), (129, 12416, 5056): (256, 192, True, 5),
    (1025, 12416, 704): (256, 256, False, 1), (450, 8320, 8128): (256, 256, False, 3), (193, 16640, 6144): (256, 256, True, 3),
    (193, 12416, 11776): (256, 256, True, 5), (129, 7168, 3008): (256, 64, False, 3),
}

# up to 64 tokens
SMALL = {
    (1, 128, 64): (128, 64, True, 1), (64, 384, 192): (128, 64, True, 1),            # one stage; a ragged last feature tile, three stages
    (64, 4096, 4096): (128, 64, True, 8), (7, 1280, 4096): (128, 64, True, 16),
    (64, 32896, 64): (256, 64, True, 1), (9, 11136, 3008): (256, 64, True, 5),       # ragged last tile
    (5, 28672, 320): (128, 64, True, 1),                                             # workgroups start at all five stages
}
