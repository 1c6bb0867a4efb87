"""Shapes of the decay front by the kernel that takes them, so that the GPU tests that take them from here test what they say (the routes are
pinned on the CPU).  Widths from 640 up give a wave two to eight blocks of channels: loads of the next block are on their way behind the
ones that a wave waits for, and every place in LDS is used again."""

# kernel and its tile: (B, T, H)
SEVERAL_BLOCKS = {
    "decay_input_split_kernel<1, 12, %s, 1>": [(2500, 1, 32), (131, 31, 12), (205, 19, 10), (2100, 1, 16), (5000, 1, 12), (257, 11, 32)],
    "decay_input_split_kernel<1, 12, %s, 2>": [(1100, 1, 32), (1500, 1, 10), (61, 33, 16)],
    "decay_input_split_kernel<1, 12, %s, 4>": [(24, 1, 32), (9, 17, 16), (1000, 1, 12), (3, 300, 10)],
    "decay_input_split_kernel<2, 8, %s, 1>": [(131, 33, 32), (5, 1531, 32), (7, 1001, 12), (131, 33, 10), (9, 900, 16)],
    "decay_input_split_kernel<4, 8, %s, 1>": [(3, 5000, 12), (131, 65, 10), (2, 5000, 32), (5, 1999, 16)],
}
# tiles of 128 tokens of one sequence: sequences shorter than a tile, of one tile and a token more
WHOLE = [(500, 50, 2), (400, 63, 2), (257, 64, 2), (255, 65, 2), (140, 127, 2), (256, 128, 2), (70, 129, 2), (500, 50, 4)]
