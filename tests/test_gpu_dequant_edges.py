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
    (5, 18944, Keep(k_keep=18931), 0),             # turns of a long row on several waves, one chunk each
    (1300, 2048, Keep(k_keep=2041), 0),            # two chunks in flight: a row of 4, of 2, of 1 chunk, narrower rows
    (2601, 1024, Keep(k_keep=1017), 0),
    (5203, 512, Keep(k_keep=511), 0),
    (9001, 384, Keep(k_keep=259), 0),
    (5201, 8192, Keep(n_keep=2100, k_keep=4099), 0),   # eight: a row of nine chunks, of five, four, three, two, one, narrower ones
    (5003, 2176, Keep(k_keep=2175), 0),
    (5001, 2048, Keep(k_keep=2043), 0),
    (6001, 1536, Keep(k_keep=1530), 0),
    (9003, 1024, Keep(k_keep=1023), 0),
    (17001, 512, Keep(k_keep=509), 0),
    (35001, 384, Keep(row_seg_stride=7, row_seg_keep=5, row_seg_limit=34993, k_keep=257), 0),
    (65539, 256, Keep(k_keep=250), 0),
    (3300, 3072, Keep(k_keep=256 * 9, col_seg_stride=12, col_seg_keep=9), 0),
    (5, 2040 * 64, Keep(k_keep=2040 * 55, col_seg_stride=64, col_seg_keep=55), 0),
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
