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
    # nothing cut, a workgroup per compute unit: each number of features with up to 80 and up to 96 token rows, one stage of k, as many as
    # their rings hold, odd and even numbers of them; ragged last feature tiles
    (65, 7168, 3584): (32, 80, True, 1), (80, 8064, 128): (32, 80, True, 1), (77, 12160, 640): (48, 80, True, 1), (66, 16256, 1664): (64, 80, True, 1),
    (72, 20352, 8064): (80, 80, True, 1), (81, 8192, 2048): (32, 96, True, 1), (96, 11136, 3456): (48, 96, True, 1), (90, 14848, 3712): (64, 96, True, 1),
    (85, 20352, 6528): (80, 96, True, 1), (79, 17024, 256): (80, 80, True, 1),
}

# up to 64 tokens
SMALL = {
    (1, 128, 64): (128, 64, True, 1), (64, 384, 192): (128, 64, True, 1),            # one stage; a ragged last feature tile, three stages
    (64, 4096, 4096): (128, 64, True, 8), (7, 1280, 4096): (128, 64, True, 16),
    (64, 32896, 64): (256, 64, True, 1), (9, 11136, 3008): (256, 64, True, 5),       # ragged last tile
    (5, 28672, 320): (128, 64, True, 1),                                             # workgroups start at all five stages
    # nothing cut: each number of features with 1 to 8 token rows, 9 to 16, 17 to 24 and 25 to 32; fewer k stages than wavefronts, as many as
    # their rings hold and a few more or less, many; a ragged last tile where the number of features allows one
    (1, 4096, 64): (16, 32, True, 1), (8, 1536, 3008): (16, 32, True, 1), (9, 3968, 2624): (16, 32, True, 1), (16, 4096, 4032): (16, 32, True, 1),
    (24, 2048, 8128): (16, 32, True, 1), (32, 4096, 1472): (16, 32, True, 1), (8, 6016, 704): (24, 32, True, 1), (15, 6016, 2112): (24, 32, True, 1),
    (17, 4224, 1024): (24, 32, True, 1), (32, 6144, 6208): (24, 32, True, 1), (3, 8064, 1984): (32, 32, True, 1), (13, 8192, 576): (32, 32, True, 1),
    (23, 8192, 1984): (32, 32, True, 1), (25, 6272, 1088): (32, 32, True, 1), (7, 12160, 3072): (48, 32, True, 1), (16, 8320, 3136): (48, 32, True, 1),
    (8, 16256, 3136): (64, 32, True, 1), (10, 12416, 3200): (64, 32, True, 1), (1, 20352, 3072): (80, 32, True, 1), (16, 16640, 3200): (80, 32, True, 1),
    (2, 24448, 3072): (96, 32, True, 1), (12, 20608, 3136): (96, 32, True, 1), (8, 28544, 3072): (112, 32, True, 1), (9, 24704, 3072): (112, 32, True, 1),
    (5, 32640, 3072): (128, 32, True, 1), (14, 28800, 3136): (128, 32, True, 1),
    # nothing cut either: each number of features with up to 48 and up to 64 token rows; one stage of k, as many as their rings hold, odd and even
    # numbers of them; ragged last feature tiles
    (33, 4096, 128): (16, 48, True, 1), (48, 3968, 3968): (16, 48, True, 1), (36, 8064, 1920): (32, 48, True, 1), (47, 8192, 2176): (32, 48, True, 1),
    (17, 12160, 2048): (48, 48, True, 1), (24, 16256, 6528): (64, 48, True, 1), (32, 20352, 896): (80, 48, True, 1), (20, 24448, 640): (96, 48, True, 1),
    (64, 8064, 640): (32, 64, True, 1), (49, 12160, 1152): (48, 64, True, 1), (63, 16256, 3072): (64, 64, True, 1), (50, 20352, 128): (80, 64, True, 1),
    (64, 24448, 2176): (96, 64, True, 1),
}
