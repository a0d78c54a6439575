"""Host-side checks of which linears the ring kernel takes (no GPU), where uniql_w4_linear_kernel tells it from the other decode-batch kernel: column
segments of 17..32 tokens."""
import pytest

import paper_2512_03383_amd as uq
from paper_2512_03383_amd import KeepDesc

RING = 8   # waves that K is split over


def ring(N, K, M, keep, ldx=None):
    c = uq.uniql_w4_linear_kernel(N, K, keep, M, ldx=ldx)
    return c[0] == 2 and c[3] == RING


@pytest.mark.parametrize("M", [17, 32])
def test_segments_of_17_tokens_and_more(M):
    seg = KeepDesc(col_seg_stride=128, col_seg_keep=108)
    assert ring(4096, 4096, M, seg) and not ring(4097, 4096, M, seg) and not ring(4096, 4224, M, seg) and not ring(4096, 4096, 33, seg)
    assert ring(4096, 2048, M, seg) and not ring(4096, 1920, M, seg)
    # (short segments of partial blocks stay with the other decode-batch kernel)
    assert not ring(1000, 3584, M, KeepDesc(col_seg_stride=32, col_seg_keep=26)) and ring(1000, 3584, M, KeepDesc(col_seg_stride=32, col_seg_keep=24))
    assert uq.uniql_w4_linear_kernel(4096, 4096, seg, M)[1:3] == (32, 16)
