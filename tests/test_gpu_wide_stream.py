"""GPU parity of the persistent streaming kernel on codes of 8, 6 and 3 bits at one token: rows of one to eight tiles, prefixes that end
anywhere, row segments of one and two families, column segments that keep whole, partial and odd units, both together, with and without
zero points, scales of both forms of the bfloat16 unpack, infinite scales behind the kept columns; against the CPU oracle on sampled
rows.  Every case says which kernel takes it; those whose groups do not divide into a row's tiles stay with the others."""
import numpy as np
import pytest

import workloads as wl
from parity_util import NORM_TOL, NORM_TOL_BF16, TOL, TOL_BF16, linear_err, normwise_err
from workloads import Keep

pytestmark = pytest.mark.gpu

CASES = [(4111, 1152, Keep(n_keep=4101, k_keep=1021)), (2600, 4096, Keep(n_keep=2573, k_keep=4001)), (3001, 2304, Keep()),
         (2304, 5120, Keep(row_seg_stride=128, row_seg_keep=118, row_seg_limit=2304, n_keep=18 * 118, k_keep=5113)),
         (2110, 8192, Keep(k_keep=8192)), (517, 8448, Keep(k_keep=8321)), (530, 12288, Keep(k_keep=12185)), (523, 18944, Keep(k_keep=14208)),
         (515, 16384, Keep()), (2570, 4096, Keep(k_keep=32 * 107, col_seg_stride=128, col_seg_keep=107)),
         (2051, 5120, Keep(k_keep=640 * 5, col_seg_stride=8, col_seg_keep=5)),
         (2100, 4992, Keep(k_keep=4985)), (517, 10240, Keep(k_keep=10201)),
         (2816, 4096, Keep(row_seg_stride=128, row_seg_keep=118, row_seg_limit=2816, n_keep=22 * 118, k_keep=4001)),
         (2900, 6144, Keep(row_seg_stride=64, row_seg_keep=54, row_seg_limit=1920, row_seg2_stride=100, row_seg2_keep=90, row_seg2_limit=2720, k_keep=6143)),
         (2051, 6144, Keep(k_keep=768 * 5, col_seg_stride=8, col_seg_keep=5)), (4099, 1024, Keep(k_keep=128 * 3, col_seg_stride=8, col_seg_keep=3)),
         (2053, 8192, Keep(k_keep=128 * 51, col_seg_stride=64, col_seg_keep=51)), (515, 16384, Keep(k_keep=128 * 107, col_seg_stride=128, col_seg_keep=107)),
         (2900, 6144, Keep(row_seg_stride=64, row_seg_keep=54, row_seg_limit=1920, row_seg2_stride=100, row_seg2_keep=90, row_seg2_limit=2720,
                           k_keep=96 * 38, col_seg_stride=64, col_seg_keep=38))]


def rows_at_a_time(case, bits):
    """What the library has to answer: rows that a wave of the walk takes at a time (0: another kernel)."""
    if case in (3, 5, 10) or (bits == 6 and CASES[case][1] <= 2048):   # 40 or 66 groups in three or five tiles; one tile of 6-bit codes
        return 0
    keep, K = CASES[case][2], CASES[case][1]
    span = K if keep.col_seg_stride else keep.k_keep or K
    return {1: 4, 2: 2}.get((span + 2047) // 2048, 1)


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("bits", [3, 6, 8])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_one_token(uref, bits, fmt, case):
    import torch
    import paper_2512_03383_amd as uq
    N, K, keep = CASES[case]
    rng = wl.rng_for(75, 100 * case + bits)
    w = wl.gen_linear8(rng, N, K, fmt=fmt) if bits == 8 else wl.gen_linear_bits(rng, N, K, bits, fmt=fmt)
    if case % 2:
        w["zeros"] = None
    s = w["scales"].view(np.uint16)
    shift = 1.0
    if fmt == "bf16" and case % 3 == 0:      # some rows with scales past where the unpack changes form
        large = rng.integers(0, 2, s.shape).astype(bool) & (np.arange(N) % 3 == 0)[:, None]
        s[large] = ((rng.integers(242, 247, s.shape) << 7) | rng.integers(0, 128, s.shape)).astype(np.uint16)[large]
        shift = 2.0 ** -10                   # (a sum stays below the largest float)
    if keep.col_seg_stride == 0 and keep.k_keep:
        s[::2, (keep.k_keep + 127) // 128:] = 0x7F80 if fmt == "bf16" else 0x7C00   # pruned groups do not count
    W = uq.QuantLinear.from_numpy(w, bits=bits)
    nk, kk = uq.kept_dims(W, keep)
    walk = rows_at_a_time(case, bits)
    assert uq.uniql_w4_linear_kernel(N, K, keep, 1, bits=bits, bf16=fmt == "bf16") == (0, int(walk > 0), walk, int(walk > 0))
    x = wl.gen_activations(rng, 1, kk, fmt=fmt)
    xd = torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda().view(torch.bfloat16 if fmt == "bf16" else torch.float16) * shift
    xn = xd.view(torch.int16).cpu().numpy().view(np.uint16 if fmt == "bf16" else np.float16)
    rows = np.unique(np.concatenate([[0, 1, 7, 8, nk // 2, nk - 2, nk - 1], rng.integers(0, nk, 120)])).astype(np.int32)
    y = torch.full((1, nk + 5), -5.0, dtype=xd.dtype, device="cuda")
    uq.uniql_w4_linear(W, keep, xd, y[:, :nk])
    torch.cuda.synchronize()
    assert torch.all(y[:, nk:] == -5.0), "wrote past n_keep"
    ref = uref.wq_linear(bits, w["qweight"], w["scales"], w["zeros"], xn, keep, fmt=fmt, rows=rows)
    got = y[:, :nk].double().cpu().numpy()[:, rows]
    assert linear_err(got, ref) <= (TOL_BF16 if fmt == "bf16" else TOL)
    assert normwise_err(got, ref) <= (NORM_TOL_BF16 if fmt == "bf16" else NORM_TOL)


# one-hot activations: every row's output is the stored weight of that column, bit for bit
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("bits", [3, 6, 8])
@pytest.mark.parametrize("N,K,keep", [(2600, 4096, Keep(k_keep=4001)), (2100, 4992, Keep()), (517, 10240, Keep(k_keep=10201)),
                                      (2570, 4096, Keep(k_keep=32 * 107, col_seg_stride=128, col_seg_keep=107)),
                                      (2051, 6144, Keep(k_keep=768 * 5, col_seg_stride=8, col_seg_keep=5))])
def test_one_hot_columns(bits, fmt, N, K, keep):
    import torch
    import paper_2512_03383_amd as uq
    rng = wl.rng_for(77, N + bits)
    w = wl.gen_linear8(rng, N, K, fmt=fmt) if bits == 8 else wl.gen_linear_bits(rng, N, K, bits, fmt=fmt)
    if N % 2:
        w["zeros"] = None
    W = uq.QuantLinear.from_numpy(w, bits=bits)
    assert uq.uniql_w4_linear_kernel(N, K, keep, 1, bits=bits, bf16=fmt == "bf16")[1] == 1
    dense = uq.uniql_w4_dequant(W, keep)
    kk = dense.shape[1]
    for k in sorted({0, 1, 7, 8, 15, 16, 31, 32, 63, 127, 128, 2047, 2048, kk - 9, kk - 2, kk - 1, *rng.integers(0, kk, 24).tolist()}):
        x = torch.zeros((1, kk), dtype=dense.dtype, device="cuda")
        x[0, k] = 1.0
        y = uq.uniql_w4_linear(W, keep, x)
        torch.cuda.synchronize()
        assert torch.equal(y[0], dense[:, k]), k
