"""Host-side checks of which kernel a linear takes (no GPU): uniql_w4_linear_kernel reports the dispatch that uniql_w4_linear
follows."""
import pytest

import paper_2512_03383_amd as uq
from paper_2512_03383_amd import KeepDesc

STREAM, STAGED, PIPE, BIG, TILED, RING = range(6)   # as reported, but the decode-batch kernel with a tile is the ring kernel


def kernel(*a, **kw):
    c = uq.uniql_w4_linear_kernel(*a, **kw)
    assert c[0] != STAGED or c[1:] == (0, 0, 0) or (c[3] == 8 and c[1] in (4, 8, 16, 32) and c[2] % 16 == 0 and c[2] >= 16)
    return RING if c[0] == STAGED and c[3] == 8 else c[0]


def seg(stride, keep):
    return KeepDesc(col_seg_stride=stride, col_seg_keep=keep)


def test_reports_without_running():
    assert uq.uniql_w4_linear_kernel(4096, 4096, None, 1) == (STREAM, 0, 0, 0)
    assert uq.uniql_w4_linear_kernel(4096, 4096, None, 8, col_interleave=32)[0] == STREAM
    assert uq.uniql_w4_linear_kernel(4096, 4096, None, 8) == (STAGED, 8, 16, 8)        # the ring kernel
    assert uq.uniql_w4_linear_kernel(14336, 4096, None, 8) == (STAGED, 0, 0, 0)        # the block-staged one
    assert uq.uniql_w4_linear_kernel(14336, 4096, None, 4096) == (BIG, 256, 256, 1)
    with pytest.raises(uq.UniqlError):
        uq.uniql_w4_linear_kernel(4096, 4100, None, 8)
    with pytest.raises(uq.UniqlError):
        uq.uniql_w4_linear_kernel(4096, 4096, KeepDesc(k_keep=4097), 8)
    with pytest.raises(uq.UniqlError):
        uq.uniql_w4_linear_kernel(4096, 4096, None, 65, col_interleave=32)
    with pytest.raises(uq.UniqlError):
        uq.uniql_w4_linear_kernel(128, 32896, None, 8, bits=8)


# column rules and sizes that neither the decode-batch kernel nor the pipelined one takes keep K split over four or eight waves
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("N,K,keep", [(4096, 4096, seg(256, 216)), (3840, 3840, seg(96, 80)), (2560, 2560, seg(80, 68)),
                                      (4096, 4096, seg(128, 107)), (4096, 896, None), (2560, 2560, KeepDesc(k_keep=5))])
def test_unusual_rules_keep_their_split_of_k(N, K, keep, bf16):
    for M in (33, 40, 48, 64):
        assert uq.uniql_w4_linear_kernel(N, K, keep, M, bf16=bf16) == (TILED, 64, 32, 4)
    if K < 1024:
        for M in (2, 8, 16):
            assert uq.uniql_w4_linear_kernel(N, K, keep, M, bf16=bf16) == (TILED, 16, 16, 8)
        for M in (17, 32):
            assert uq.uniql_w4_linear_kernel(N, K, keep, M, bf16=bf16) == (TILED, 32, 16, 8)


@pytest.mark.parametrize("K,keep,first", [(896, None, 2), (4096, seg(256, 216), 9), (4096, seg(128, 107), 9)])
def test_tall_matrices_of_unusual_rules(K, keep, first):
    for M, want in ((first, (TILED, 16, 64, 4)), (16, (TILED, 16, 64, 4)), (17, (TILED, 32, 64, 4)), (32, (TILED, 32, 64, 4)),
                    (33, (TILED, 64, 64, 4)), (64, (TILED, 64, 64, 4))):
        assert uq.uniql_w4_linear_kernel(12288, K, keep, M) == want, M


# decode batches of 2..8 tokens are one kernel's up to 600 row tiles, so that q, k and v share a launch
@pytest.mark.parametrize("N", [1024, 6400, 8192, 9472, 18944])
@pytest.mark.parametrize("K,keep", [(4096, None), (8192, None), (4096, seg(128, 108))])
def test_small_decode_batches_share_one_kernel(N, K, keep):
    for M in (2, 5, 8):
        assert kernel(N, K, keep, M) == (RING if N <= 9600 else STAGED)
    assert kernel(N, 8192, keep and seg(128, 108), 12) == (RING if N < 6400 else PIPE)


# columns behind the last whole block of eight cost the tiled kernels more than the pipelined one (65 against 39 us at 2560 x 1999
# and 2048 tokens), whole blocks nothing
def test_odd_columns_of_prompts():
    assert uq.uniql_w4_linear_kernel(2560, 2560, KeepDesc(k_keep=1999), 2048, ldx=1999)[0] == PIPE
    for bf16 in (False, True):
        for M in (333, 777, 1000, 1500):
            assert uq.uniql_w4_linear_kernel(4096, 14336, KeepDesc(k_keep=9318), M, bf16=bf16)[0] == PIPE, M
    assert uq.uniql_w4_linear_kernel(14336, 4096, KeepDesc(n_keep=12185), 4096)[0] == BIG


# codes of 8, 6 and 3 bits: few rows or very few tokens stay with the streaming kernels (a token per grid row)
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("bits", [8, 6, 3])
def test_wide_codes_stream_where_that_is_faster(bits, bf16):
    def route(N, K, M, keep=None):
        return kernel(N, K, keep, M, bits=bits, bf16=bf16)
    for K in (1024, 4096, 14336):
        for M in (2, 4, 8):
            assert route(256, K, M) == STREAM
    assert route(1024, 1024, 2) == STREAM and route(1024, 4096, 2) == STREAM
    assert route(2048, 14336, 2) == STREAM
    for N, K in ((4096, 4096), (12185, 4096), (4096, 14336)):
        for M in (8, 16, 48, 512):
            assert route(N, K, M) == (RING if M <= 16 else PIPE)
    if bits == 6 and not bf16:
        for N, K in ((4096, 4096), (4096, 14336), (14336, 2048)):
            assert route(N, K, 2) == RING
    assert route(128, 896, 8) == STREAM


# what a grid holds: 65535 token tiles in y, fewer than 2^32 threads in all
@pytest.mark.parametrize("N,K,keep,M,bits", [
    (100, 4096, seg(256, 216), 5_000_000, 4), (16, 1024, KeepDesc(k_keep=5), 7_000_000, 4), (100, 896, None, 3_000_000, 4),
    (1_000_000, 1024, None, 65535, 8), (2_000_000, 1024, None, 65535, 8), (500_000, 1024, seg(64, 54), 100_000, 4),
    (4_000_000, 1024, None, 65_000, 4), (128256, 4096, None, 65535, 3)])
def test_grids_hold_the_largest_calls(N, K, keep, M, bits):
    kernel, bm, bn, _ = uq.uniql_w4_linear_kernel(N, K, keep, M, bits=bits)
    if kernel == PIPE:
        assert -(-N // bn) * -(-M // bm) * 768 < 2 ** 32
    elif kernel == TILED:
        assert -(-M // bm) <= 65535


# the sizes of the GPU parity tests take every tile that the pipelined kernel is built with
@pytest.mark.parametrize("segments", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("bits", [4, 8, 6, 3])
def test_parity_sizes_take_every_tile(bits, bf16, segments):
    import pipe_shapes as ps
    seen = set()
    for i, (N, K, M) in enumerate(ps.SIZES):
        choice = uq.uniql_w4_linear_kernel(N, K, ps.keep_rule(N, K, segments), M, bits=bits, bf16=bf16,
                                           ldx=ps.kept_columns(K, segments) + i % 3)
        if choice[0] == PIPE:
            seen.add(choice[1:])
    assert seen == ps.tiles(bits, segments)


# 33..64 tokens of 8, 6 and 3 bits: K over four groups while one round of those tiles takes the matrix, then 64 or 96 rows x all tokens
@pytest.mark.parametrize("bits,last", [(8, 256), (6, 256), (3, 512)])
def test_height_at_which_wide_codes_change_their_split(bits, last):
    for K in (2560, 4096):
        for M in (40, 64):
            assert uq.uniql_w4_linear_kernel(16 * last, K, None, M, bits=bits)[1] == 32
            assert uq.uniql_w4_linear_kernel(16 * last + 1, K, None, M, bits=bits)[1] in (48, 64)


# decode batches of 17..32 tokens on column segments of more than 256 row tiles, and of 9..32 tokens on long rows from 400 row tiles on, go to the
# pipelined kernel; the others are the ring kernel's, so that they share a launch (6000 + 1536 rows x 2560 columns at 9 tokens 8.1 us, 13.6 in two)
@pytest.mark.parametrize("bf16", [False, True])
def test_decode_batches_that_the_pipelined_kernel_takes(bf16):
    for N, K, keep in ((512, 4096, seg(128, 96)), (2560, 5120, seg(64, 54)), (4096, 4096, seg(128, 108)), (4112, 4096, seg(128, 108))):
        late = PIPE if N > 4096 else RING
        for M, want in ((8, RING), (16, RING), (17, late), (32, late)):
            assert kernel(N, K, keep, M, bf16=bf16) == want, (N, M)
    for N, want in ((5985, RING), (6384, RING), (6385, PIPE)):
        for M in (9, 17, 32):
            assert kernel(N, 8192, None, M, bf16=bf16) == want
        assert kernel(N, 8192, None, 8, bf16=bf16) == RING


# column segments of 17..32 tokens: the ring kernel up to 64 groups (more than 192 row tiles: up to 24 tokens), up to 96 where the block-staged one is not the
# better; where that is better than the pipelined one, segments whose kept columns are not whole blocks of eight in long rows stay with it (512
# x 14208, 98 of 128 columns, 17 tokens: 0.82 of the other kernel's time): fp16, or segments of fewer than 64 columns
@pytest.mark.parametrize("M", [17, 32])
def test_segments_that_decode_batches_keep(M):
    for N, K, keep, f16, bf in ((512, 14208, seg(128, 98), STAGED, PIPE), (512, 14208, seg(128, 96), PIPE, PIPE), (1024, 4096, seg(64, 54), RING, RING),
                                (1024, 4224, seg(64, 54), RING, RING), (3000, 8192, seg(64, 54), RING, RING), (3584, 7936, seg(64, 54), *[RING if M == 17 else PIPE] * 2),
                                (3584, 8192, seg(64, 54), *((RING, RING) if M == 17 else (STAGED, PIPE))), (2560, 10624, seg(128, 108), STAGED, RING),
                                (3072, 12288, seg(128, 96), RING, RING), (3073, 12288, seg(128, 96), PIPE, PIPE), (3072, 12416, seg(128, 96), PIPE, PIPE),
                                (1000, 4224, seg(32, 26), STAGED, STAGED), (1000, 4224, seg(32, 24), RING, RING),
                                (4097, 14208, seg(64, 54), PIPE, PIPE), (1000, 3456, seg(32, 26), RING, RING), (1000, 3584, seg(32, 26), STAGED, STAGED)):
        for bf16, want in ((False, f16), (True, bf)):
            assert kernel(N, K, keep, M, bf16=bf16) == want, (N, K, bf16)


# one token of 8-, 6- and 3-bit codes: the walk's rows at a time, and what it leaves to the other kernels
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("bits", [8, 6, 3])
def test_one_token_of_wide_codes(bits, bf16):
    def rows(N, K, keep=None):
        c = uq.uniql_w4_linear_kernel(N, K, keep, 1, bits=bits, bf16=bf16)
        assert c[0] == STREAM and c[1] == c[3] == int(c[2] > 0)
        return c[2]
    for N, K, want in ((4096, 1024, 0 if bits == 6 else 4), (4095, 1024, 0), (2560, 4096, 2), (2559, 4096, 0), (2048, 6144, 1), (2047, 6144, 0), (2048, 8192, 1),
                       (512, 10240, 1), (511, 10240, 0), (512, 16384, 1), (4096, 5120, 0), (4096, 8448, 0), (4096, 16512, 0)):
        assert rows(N, K) == want, (N, K)
    assert rows(4096, 8192, KeepDesc(k_keep=4096)) == 2 and rows(4096, 5120, KeepDesc(k_keep=4096)) == 2
    assert rows(4096, 4096, KeepDesc(k_keep=7)) == 0
    assert rows(4096, 6144, seg(8, 5)) == 1 and rows(4096, 6144, seg(24, 5)) == 1 and rows(4096, 6144, seg(12, 5)) == 0
    assert rows(4096, 4096, KeepDesc(row_seg_stride=64, row_seg_keep=40, row_seg_limit=4096)) == 2
    assert rows(4096, 4096, KeepDesc(row_seg_stride=64, row_seg_keep=39, row_seg_limit=4096)) == 0


# column segments: tiles of 128 tokens wherever the cost of a launch says so, from one token tile on (16384 x 4096, 108 of 128 columns,
# 256 tokens: 52 -> 41 us)
@pytest.mark.parametrize("bits", [4, 8, 6, 3])
def test_tall_segments_take_128_tokens(bits):
    assert uq.uniql_w4_linear_kernel(16384, 4096, seg(128, 108), 256, bits=bits)[:3] == (PIPE, 128, 128)
    assert uq.uniql_w4_linear_kernel(24576, 4096, seg(128, 108), 128, bits=bits)[:3] == (PIPE, 128, 128)
    assert uq.uniql_w4_linear_kernel(4096, 4096, seg(128, 108), 256, bits=bits)[:3] == (PIPE, 64, 64)
