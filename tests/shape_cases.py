"""Sizes of the GPU tests that are written for one launch plan, each with the plan it is there for (not collected by
pytest).  test_launch_plan.py asks the library's plans on the host whether the sizes still get them: a cost constant
that is fitted again must not empty a test."""
FOLDED, LONGEST_FIRST = 0, 1

# forward of 64 rows: (S, heads); one row, one block of 32 rows, one more, all but one in the last tile
FWD_64_EDGES = [(257, 48), (288, 48), (289, 48), (319, 48)]

# backward of 32 rows: one tile and its neighbours, waves without a tile, a ragged last tile behind a whole sweep
BWD_32_EDGES = [(S, 3) for S in (31, 32, 33, 257, 1000)]

# whole 32-row tiles: (S, heads, keys of a streamed tile) -> rows and order of the forward
FWD_SHAPES = {(288, 9, 32): (32, LONGEST_FIRST), (320, 48, 32): (64, LONGEST_FIRST), (352, 48, 64): (128, LONGEST_FIRST),
              (704, 160, 64): (256, LONGEST_FIRST), (704, 100, 64): (256, FOLDED)}

# ragged lengths: (S, heads) -> rows, joint launch, orders of dK/dV and of dQ
BWD_SHAPES = {(300, 3): (32, 1, LONGEST_FIRST, LONGEST_FIRST), (1000, 4): (32, 1, LONGEST_FIRST, LONGEST_FIRST),
              (353, 48): (64, 1, LONGEST_FIRST, LONGEST_FIRST), (513, 64): (128, 1, LONGEST_FIRST, LONGEST_FIRST),
              (700, 160): (256, 1, LONGEST_FIRST, LONGEST_FIRST)}

# the same for the longer sequences that work 256 rows, an even and an odd number of tiles
BWD_LONG_SHAPES = {(8155, 16): (256, 0, FOLDED, FOLDED), (7773, 48): (256, 0, FOLDED, FOLDED), (5799, 64): (256, 0, LONGEST_FIRST, FOLDED),
                   (5611, 64): (256, 0, LONGEST_FIRST, LONGEST_FIRST),
                   (4248, 20): (256, 1, LONGEST_FIRST, LONGEST_FIRST)}

# projection: (rows of the tensor, K, N, first row) -> tokens and features of a tile; several tiles for a workgroup where more than 256
LINEAR_SHAPES = {(65, 128, 128, 0): (64, 64), (257, 384, 384, 1): (64, 64), (700, 640, 640, 3): (64, 64), (3261, 128, 640, 5): (64, 64),
                 (900, 5120, 1920, 0): (128, 64), (3501, 384, 384, 1): (128, 64),
                 (2500, 256, 896, 0): (128, 128), (5000, 384, 640, 7): (128, 128), (9290, 128, 896, 5): (128, 128),
                 (9000, 128, 1152, 0): (192, 128), (21837, 128, 384, 2): (192, 128),
                 (17003, 256, 384, 3): (256, 128), (32879, 128, 384, 0): (256, 128),
                 (40001, 384, 640, 130): (256, 256)}

# workgroups of 256 rows: the last tile of one row, of one 64-row wave and its neighbours, of two waves and a ragged third, whole;
# (S, heads) -> order of the forward: in eight waves of 32 rows, and in four of 64
FWD_LONG_EDGES = {(513, 128): FOLDED, (575, 160): LONGEST_FIRST, (576, 128): FOLDED, (577, 160): LONGEST_FIRST, (705, 100): FOLDED, (769, 128): FOLDED,
                  (1024, 160): LONGEST_FIRST, (1025, 80): FOLDED}
FWD_FOUR_WAVE_EDGES = {(3329, 48): LONGEST_FIRST, (3391, 48): LONGEST_FIRST, (3521, 48): LONGEST_FIRST, (3584, 60): LONGEST_FIRST,
                       (3329, 72): FOLDED, (3391, 68): FOLDED, (3392, 68): FOLDED, (3393, 68): FOLDED, (3585, 64): FOLDED}
# (S, heads) -> orders of dK/dV and of dQ, in four waves
BWD_LONG_EDGES = {(3841, 160): (FOLDED, FOLDED), (3903, 128): (FOLDED, FOLDED), (3904, 128): (FOLDED, FOLDED), (3905, 128): (FOLDED, FOLDED),
                  (4351, 96): (LONGEST_FIRST, LONGEST_FIRST), (4352, 96): (LONGEST_FIRST, LONGEST_FIRST), (5121, 160): (LONGEST_FIRST, FOLDED)}

# (S, heads): both gradients in one launch of four waves, the last tile of one row, of one wave and its neighbours, whole
BWD_JOINT_EDGES = [(3073, 24), (3329, 20), (3391, 20), (3392, 20), (3393, 20), (3584, 20), (3585, 24)]

# row sums of a long sweep: (S, heads) -> order of the forward
FWD_LONG_SUMS = {(16384, 16): FOLDED}

# batches in one packed buffer: (B, S, heads) -> orders of dK/dV and of dQ; the forward works 256 rows too
LONG_LAYOUTS = {(2, 3905, 64): (FOLDED, FOLDED), (3, 4351, 32): (LONGEST_FIRST, LONGEST_FIRST)}

# fp32 on fp16 matrix instructions, forward and backward: (S, heads, d); a last tile of one row, of all but one, whole, and of 17; sweeps of several steps a wave
F32_SPLIT_EDGES = [(1057, 8, 64), (1055, 8, 64), (1056, 8, 64), (1073, 8, 64), (865, 8, 128), (895, 8, 128), (896, 8, 128), (881, 8, 128), (2049, 3, 64), (2047, 3, 128)]
F32_SPLIT_ONE = [(1300, 4, 128), (1600, 4, 64)]
