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


# (bits, K, N, M, segments, tokens of a tile): grids whose last round goes out as halves of its tiles; in those with at most half a tile of tokens left over
# (8170 x 1170, 23680 and 19027 x 700, 5068 x 777) second halves have no token.  Codes of 8 bits in 128-token tiles are also brought into the L2 ahead.
HALVES = [(8, 1024, 6102, 1000, False, 128), (8, 1024, 6102, 1000, True, 128), (8, 1024, 8170, 1170, False, 128), (8, 1024, 8170, 1170, True, 128), (8, 1152, 12185, 500, False, 128),
          (6, 1024, 8170, 1170, False, 128), (6, 1024, 8170, 1170, True, 128), (6, 1024, 5068, 777, False, 96), (6, 1024, 5068, 777, True, 96)]
HALVES += [(bits, *size) for bits in (4, 3) for size in ((1024, 11789, 1500, False, 128), (1024, 23680, 700, False, 128), (1024, 16442, 1500, True, 128), (1024, 19027, 700, True, 128),
                                                         (1024, 5068, 777, False, 96), (1024, 5068, 777, True, 96))]


def halves_rule(K, N, segments):
    """The rule of a case of HALVES: all rows but three, 102 of 128 columns or all but thirteen."""
    return dict(n_keep=N - 3, k_keep=K // 128 * 102, col_seg_stride=128, col_seg_keep=102) if segments else dict(n_keep=N - 3, k_keep=K - 13)


def half_tiles(rows, M, tile, cus=256):
    """Tiles of a grid that go out as halves, and all of them, for a tile of (tokens, rows)."""
    tiles = -(-rows // tile[1]) * -(-M // tile[0])
    rest = tiles % cus
    return (rest if tiles > cus and 2 * rest <= cus else 0), tiles
