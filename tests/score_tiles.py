"""Shapes that take each kernel of the scoring's partial sums: every stride,
causal and not, in every tile size, each with more than one row tile and,
where the 128 / stride rows of a block allow it, a ragged last one.
tests/test_dispatch_host.py checks that each shape takes the tile named here."""

CUS = 256  # compute units that the shapes below are for

# (stride, causal, rows of the tile, query heads, blocks)
CASES = [
    (1, True, 256, 2, 23), (1, True, 128, 2, 11), (1, True, 64, 2, 9), (1, True, 32, 2, 3),
    (1, False, 256, 2, 17), (1, False, 128, 2, 9), (1, False, 64, 2, 7), (1, False, 32, 2, 3),
    (2, True, 256, 2, 45), (2, True, 128, 2, 23), (2, True, 64, 2, 17), (2, True, 32, 2, 3),
    (2, False, 256, 2, 33), (2, False, 128, 2, 17), (2, False, 64, 2, 11), (2, False, 32, 2, 3),
    (4, True, 256, 2, 89), (4, True, 128, 2, 43), (4, True, 64, 2, 31), (4, True, 32, 2, 3),
    (4, False, 256, 2, 65), (4, False, 128, 2, 33), (4, False, 64, 2, 23), (4, False, 32, 2, 3),
    (8, True, 256, 2, 177), (8, True, 128, 2, 85), (8, True, 64, 2, 61), (8, True, 32, 2, 3),
    (8, False, 256, 2, 129), (8, False, 128, 4, 41), (8, False, 64, 2, 43), (8, False, 32, 2, 3),
    (16, True, 256, 52, 49), (16, True, 128, 68, 17), (16, True, 64, 88, 9), (16, True, 32, 2, 5),
    (16, False, 256, 60, 33), (16, False, 128, 4, 81), (16, False, 64, 2, 85),
    (16, False, 32, 2, 5), (32, True, 256, 52, 97), (32, True, 128, 68, 33),
    (32, True, 64, 88, 17), (32, True, 32, 2, 9), (32, False, 256, 60, 65),
    (32, False, 128, 44, 33), (32, False, 64, 26, 33), (32, False, 32, 2, 9),
    (64, True, 256, 52, 193), (64, True, 128, 68, 65), (64, True, 64, 88, 33),
    (64, True, 32, 2, 17), (64, False, 256, 60, 129), (64, False, 128, 44, 65),
    (64, False, 64, 26, 65), (64, False, 32, 2, 17),
]
