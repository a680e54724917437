"""Sizes that GPU tests use because of the kernel that serves them.  test_dispatch_rules.py checks on the CPU that the
library's rules still send them there, so that a change of a rule cannot quietly take a kernel's tests away."""

# Linear layers: (R, K, F), then the tiles (columns) of y, grad x and grad W and whether grad W leaves partial sums.  Between
# them every tile of every product, each with a contraction that ends in half a tile (or, grad W, in a ragged one), a ragged
# last row tile and a ragged last column tile behind a whole one.
LINEAR = [
    ((1, 96, 224), (64, 64, 64), False),
    ((1, 480, 3232), (64, 64, 128), False),
    ((214, 96, 96), (64, 64, 64), True),
    ((4709, 288, 224), (128, 128, 128), True),
    ((8243, 224, 288), (192, 192, 128), True),
    ((4100, 224, 1568), (256, 128, 128), True),
    ((3890, 1632, 544), (192, 256, 192), True),
    ((3114, 4192, 288), (64, 256, 256), True),
]

# The 256-row tiles: (R, K, F), the tiles of y, grad x and grad W.  One contraction tile and half of one, one and a half, two;
# a last row tile of one row, of all but one; a last column tile of one block of 32; several output tiles per workgroup with
# contractions shorter than the loads run ahead; grad W with the border between the two row sets inside a part.
LINEAR_PIPE = [
    ((4097, 32, 1184), (192, 64, 64)),
    ((8191, 64, 416), (192, 64, 64)),
    ((33025, 32, 128), (192, 64, 64)),
    ((5000, 96, 800), (192, 64, 128)),
    ((4097, 32, 1568), (256, 64, 64)),
    ((8191, 64, 800), (256, 64, 64)),
    ((33025, 32, 224), (256, 64, 64)),
    ((5000, 96, 2592), (256, 64, 128)),
    ((33025, 96, 160), (192, 128, 64)),
    ((6145, 608, 352), (192, 192, 128)),
    ((12289, 768, 800), (192, 192, 192)),
    ((3001, 4640, 1184), (192, 256, 192)),
    ((2049, 1184, 4640), (192, 192, 256)),
]

# The 256-row tiles with row pitches other than the widths: both of them in every product
LINEAR_PITCHED = [
    ((4097, 608, 1568), (256, 192, 192)),
    ((12289, 768, 800), (192, 192, 192)),
    ((3001, 4640, 1184), (192, 256, 192)),
    ((2049, 1184, 4640), (192, 192, 256)),
]

# Forward: heads, M, N.  Eight waves on 256 rows (512 keys and more, more than 128 queries, head dims up to 96), with a whole and
# with a ragged last key tile, workgroups whose upper waves hold no row, M != N either way round
FORWARD_EIGHT_WAVES = [(33, 512, 512), (33, 513, 513), (32, 543, 543), (17, 1000, 1000), (60, 257, 512), (52, 300, 543), (25, 700, 600),
                       (28, 600, 700), (25, 1000, 2050)]
FORWARD_EIGHT_WAVES_DIMS = [8, 24, 32, 40, 64, 72, 96]
# Four waves on 128 rows, from 128 keys on (fewer keys: any call)
FORWARD_FOUR_WAVES = [(65, 130, 129), (33, 256, 250), (130, 64, 200), (33, 250, 511), (130, 128, 600)]
FORWARD_FOUR_WAVES_DIMS = [8, 24, 32, 40, 64, 72, 96, 104, 128]
FORWARD_FOUR_WAVES_WIDE = [(35, 512, 512), (25, 700, 600), (17, 1000, 1030)]   # head dims above 96, also with 512 keys and more
# On both sides of the lines of the forward for few rows: heads, M, N, d, and whether it takes the call
FORWARD_LINES = [
    (8, 1024, 128, 72, True), (8, 1025, 128, 72, False), (8, 1024, 127, 72, False), (8, 1020, 511, 96, True), (8, 1030, 511, 96, False),
    (16, 1024, 512, 40, True), (16, 1025, 512, 40, False), (16, 1024, 2047, 64, True), (16, 1025, 2047, 64, False),
    (24, 1024, 2048, 64, True), (24, 1025, 2048, 64, False), (16, 1024, 2048, 104, True), (16, 1025, 2048, 104, False),
]

# Gate: B, T, C, dtype: more partial rows than the end kernel fetches itself
GATE_MANY_ROWS = [(1, 257, 1152, "bf16"), (1, 1024, 1152, "bf16"), (3, 700, 72, "bf16"), (1, 2048, 1024, "f32"), (5, 300, 4, "f32")]
