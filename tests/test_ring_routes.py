"""Host-side checks of which linears the ring kernel takes (no GPU): column segments of 17..32 tokens, and codes of 8, 6 and 3 bits."""
import pytest

import paper_2512_03383_amd as uq
from paper_2512_03383_amd import KeepDesc

RING = 8   # waves that K is split over


def ring(N, K, M, keep, ldx=None, bits=4, bf16=False):
    c = uq.uniql_w4_linear_kernel(N, K, keep, M, ldx=ldx, bits=bits, bf16=bf16)
    return c[0] == 1 and c[3] == RING


@pytest.mark.parametrize("M", [17, 32])
def test_segments_of_17_tokens_and_more(M):
    seg = KeepDesc(col_seg_stride=128, col_seg_keep=108)
    assert ring(4096, 4096, M, seg) and not ring(4097, 4096, M, seg) and ring(4096, 4224, M, seg) == (M <= 24) and not ring(4096, 4096, 33, seg)
    assert ring(3072, 8192, M, seg) and not ring(3072, 8320, M, seg) and ring(3072, 8320, M, KeepDesc(col_seg_stride=128, col_seg_keep=104))
    assert ring(4096, 2048, M, seg) and not ring(4096, 1920, M, seg)
    # (short segments of partial blocks stay with the other decode-batch kernel)
    assert not ring(1000, 3584, M, KeepDesc(col_seg_stride=32, col_seg_keep=26)) and ring(1000, 3584, M, KeepDesc(col_seg_stride=32, col_seg_keep=24))
    assert uq.uniql_w4_linear_kernel(4096, 4096, seg, M)[1:3] == (32, 16)


@pytest.mark.parametrize("bits", [8, 6, 3])
def test_wide_codes(bits):
    def takes(N, K, M):
        return ring(N, K, M, None, bits=bits)
    assert takes(2048, 2048, 8) and takes(2048, 2304, 32) and not takes(2048, 2304, 33) and not takes(2048, 1920, 8)
    assert takes(2048, 2048, 17) and takes(2048, 2176, 17) and takes(16384, 2176, 32) == (bits != 3)
    assert takes(4096, 4096, 32) and takes(4096, 4224, 8) and takes(4096, 5120, 8) and takes(4096, 5248, 24) and takes(1024, 5120, 17) and takes(2048, 4608, 32)
    assert takes(3072, 8192, 32) and takes(3088, 8192, 25) and takes(4096, 8192, 32)
    assert takes(4112, 4096, 8) == takes(8192, 10240, 24) == (bits == 6) and not takes(8192, 10368, 17) and takes(8208, 10368, 17)
    assert takes(12288, 4096, 8) and takes(12304, 4096, 8) == takes(16384, 4096, 8) == (bits != 3) and takes(16385, 4096, 8)
    assert takes(24576, 4096, 8) and not takes(24577, 4096, 8)
    # few outputs: a token per grid row
    assert not takes(256, 4096, 8) and not takes(2048, 8192, 2) and not takes(1024, 4096, 4) and takes(1025, 8192, 4) and takes(520, 8192, 8)
    assert takes(2064, 8192, 2)


# tall prefixes of short rows: not where the ring kernel would have four fragments a block
@pytest.mark.parametrize("M", [9, 16, 17, 32])
def test_tall_prefixes(M):
    assert ring(12288, 4096, M, None) and not ring(12289, 4096, M, None) and not ring(16384, 4096, M, None) and ring(16385, 4096, M, None)
    assert ring(24576, 4096, M, None) and not ring(24577, 4096, M, None) and not ring(16385, 4224, M, None)


# up to 8 tokens: prefixes that the block-staged kernel cannot hold whole, rows of fewer than sixteen groups and some longer ones, up to three rounds of the compute units; from
# five tokens on also long rows beyond five
@pytest.mark.parametrize("M", [2, 4, 5, 8])
def test_tall_prefixes_of_few_tokens(M):
    assert ring(10224, 4096, M, None) and not ring(10225, 4096, M, None) and ring(10225, 4224, M, None) and ring(12288, 4224, M, None)
    assert ring(12288, 1920, M, None) and not ring(12289, 1920, M, None)
    for K in (2048, 2560, 2688, 4096):   # two of five tokens and more, bfloat16, at most 20 groups
        for bf16 in (False, True):
            assert ring(10225, K, M, None, bf16=bf16) == ring(12288, K, M, None, bf16=bf16) == ((M > 4) + bf16 + (K <= 2560) >= 2) and not ring(12289, K, M, None, bf16=bf16)
    assert not ring(12289, 4224, M, None) and not ring(16384, 5248, M, None) and not ring(16385, 8192, M, None) and not ring(20480, 8192, M, None)
    assert ring(20481, 4224, M, None) == ring(24576, 8192, M, None) == (M > 4) and not ring(24577, 8192, M, None) and not ring(20481, 4096, M, None)
    assert ring(9600, 8192, M, KeepDesc(col_seg_stride=128, col_seg_keep=108)) and not ring(9601, 8192, M, KeepDesc(col_seg_stride=128, col_seg_keep=108))


# 4-bit prefixes from eight groups on (one for every wave), of one row from sixteen; segments and other widths from sixteen
@pytest.mark.parametrize("M", [2, 16, 32])
def test_shortest_rows(M):
    assert ring(2048, 1024, M, None) and not ring(2048, 896, M, None) and ring(2048, 2048, M, KeepDesc(k_keep=897)) and not ring(2048, 2048, M, KeepDesc(k_keep=896))
    assert ring(2, 1024, M, None) and not ring(1, 1920, M, None) and not ring(7, 1920, M, KeepDesc(n_keep=1)) and ring(1, 2048, M, None)
    assert not ring(2048, 1920, M, KeepDesc(col_seg_stride=128, col_seg_keep=104)) and ring(2048, 2048, M, KeepDesc(col_seg_stride=128, col_seg_keep=104))
    assert not ring(3000, 1920, M, None, bits=8) and ring(3000, 2048, M, None, bits=8)


# 9 to 16 tokens: not one round of the pipelined kernel's 32-row tiles, 400 to 512 row tiles, with rows of more than 20 groups, two of which are slower here in a launch
@pytest.mark.parametrize("M", [9, 16, 17, 32])
def test_one_round_of_the_pipelined_kernel(M):
    for N, K in ((6384, 4096), (6385, 2560), (8192, 2560), (8193, 2688), (8193, 4096)):
        assert ring(N, K, M, None)
    for N, K in ((6385, 2688), (7168, 4096), (8192, 4096), (8192, 3072)):
        assert ring(N, K, M, None) == (M > 16) and ring(N, K, 8, None)
