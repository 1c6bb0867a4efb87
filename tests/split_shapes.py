"""Shapes around the split that the prefill entry points make by themselves.  The plans are pinned on the CPU (the plan's own check
and the kernels that a call launches), so that the GPU tests that take their shapes from here test what they say."""

# (B, T, H): (segments, tokens of a segment)
SPLIT = {
    (1, 898, 1): (5, 192),          # a last segment of exactly the 130 tokens of the hand-over
    (1, 1090, 2): (7, 160),         # the same, after other lengths were tried
    (1, 899, 4): (5, 192),          # one token more
    (1, 960, 64): (4, 256),         # one workgroup per compute unit
    (1, 1216, 85): (3, 416),        # most units that still split, fewest tokens
    (5, 1531, 12): (4, 384),        # ragged last chunk
    (1, 4098, 1): (13, 320),        # one unit
    (1, 2560, 16): (16, 160),       # most segments for its units
    (1, 3000, 3): (12, 256),
    (1, 4200, 32): (8, 544),        # 17 chunks a segment: two or three for each wave of the state pass
    (2, 1300, 40): (3, 448),        # 14 chunks: one or two
    (2, 1100, 40): (3, 384),        # three segments of 80 units
    (5, 1050, 16): (3, 352),
}
# left whole: too little saved (four segments of 224 tokens; three, with more than 80 units), or one unit too many for a third segment
WHOLE = [(1, 831, 4), (1, 863, 4), (1, 1215, 85), (1, 961, 85), (7, 1100, 12), (1, 4096, 86)]
