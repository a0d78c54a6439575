"""Sizes that between them take every tile of csrc/pipe_kernel.h, for the GPU parity tests and for the host check that they do."""
from paper_2512_03383_amd import KeepDesc

# (rows, stored columns, tokens): ragged in each; enough groups that every ring of slabs goes round (9 slabs of four groups, 17 of two,
# 17 of one)
SIZES = [(6410, 4224, 11), (8300, 4224, 11), (6410, 4224, 19), (8300, 4224, 19), (3000, 4224, 13), (3000, 4224, 27),
         (6410, 4224, 37), (8300, 4224, 37), (16500, 4224, 37), (6410, 4224, 51), (8300, 4224, 51), (16500, 4224, 51),
         (24700, 4224, 11), (24700, 4224, 19),   # (more rows than the ring kernel takes)
         (300, 2176, 67), (8300, 2176, 67), (11000, 2176, 67), (16500, 2176, 67), (16500, 2176, 101), (16500, 2176, 127), (5101, 2176, 333)]


def keep_rule(N, K, segments):
    """A row prefix and a prefix that ends inside a block of eight with an odd number of columns; or column segments."""
    if segments:
        return KeepDesc(n_keep=N - 3, col_seg_stride=128, col_seg_keep=102)
    return KeepDesc(n_keep=N - 3, k_keep=K - 13)


def kept_columns(K, segments):
    return K // 128 * 102 if segments else K - 13


def tiles(bits, segments):
    """(tokens, rows, waves along K) of every tile that the kernel is built with for a width and a kind of column rule."""
    narrow = bits <= 4
    t = {(16, 32, 4), (32, 32, 4), (48, 64, 4), (48, 96, 4), (64, 64, 4), (96, 128, 2), (64, 128, 2), (64, 64, 2), (128, 128, 2)}
    if narrow:
        t |= {(16, 64, 4), (32, 64, 4), (64, 96, 4), (112, 128, 2)}
    return t
