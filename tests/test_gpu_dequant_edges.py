"""Bit-exact 4-bit dequantisation where a wave's turn over a row ends: rows of 63..66, 255..258 and 511..514 words, rows whose output
starts at every 2-byte alignment, segments of whole and of partial words, head-interleaved words, more rows than
one turn of the grid; nothing is written past the last element."""
import numpy as np
import pytest

import workloads as wl
from workloads import Keep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("N,K,keep,heads", [
    (5, 128, Keep(k_keep=7), 0),
    (9, 128, Keep(k_keep=8), 0),
    (7, 128, Keep(n_keep=5, k_keep=9), 0),
    (6, 512, Keep(k_keep=503), 0),
    (6, 640, Keep(k_keep=513), 0),
    (5, 640, Keep(k_keep=527), 0),
    (9, 2048, Keep(k_keep=2033), 0),
    (9, 2048, Keep(), 0),
    (9, 2176, Keep(n_keep=8, k_keep=2049), 0),
    (3, 2176, Keep(k_keep=2063), 0),
    (5, 4096, Keep(k_keep=4081), 0),
    (5, 4096, Keep(), 0),
    (5, 4224, Keep(n_keep=4, k_keep=4097), 0),
    (6, 4224, Keep(k_keep=4111), 0),
    (4, 2048, Keep(k_keep=64 * 1, col_seg_stride=32, col_seg_keep=1), 0),
    (5, 2048, Keep(k_keep=16 * 127, col_seg_stride=128, col_seg_keep=127), 0),
    (5, 2176, Keep(k_keep=64 * 33, col_seg_stride=34, col_seg_keep=33), 0),
    (5, 2176, Keep(k_keep=16 * 109, col_seg_stride=136, col_seg_keep=109), 0),
    (262147, 128, Keep(k_keep=3), 0),              # more rows than one turn of the grid
    (5, 2048, Keep(k_keep=16 * 109, col_seg_stride=128, col_seg_keep=109), 16),
    (5, 2048, Keep(k_keep=32 * 40, col_seg_stride=64, col_seg_keep=40), 32),
])
def test_row_edges(uref, N, K, keep, heads, fmt):
    import torch
    import paper_2512_03383_amd as uq
    w = wl.gen_linear(wl.rng_for(41, N + K + heads), N, K, fmt=fmt)
    ref = uref.w4_dequant(w["qweight"], w["scales"], w["zeros"], keep, fmt=fmt).view(np.uint16)
    qw = uq.QuantLinear.from_numpy(w)
    if heads:
        qw = uq.uniql_w4_interleave(qw, heads)
    nk, kk = uq.kept_dims(qw, keep)
    buf = torch.full((nk * kk + 16,), 21.0, dtype=torch.bfloat16 if fmt == "bf16" else torch.float16, device="cuda")
    got = uq.uniql_w4_dequant(qw, keep, out=buf[:nk * kk].view(nk, kk))
    torch.cuda.synchronize()
    assert np.array_equal(got.view(torch.int16).cpu().numpy().view(np.uint16), ref)
    assert torch.all(buf[nk * kk:] == 21.0)
