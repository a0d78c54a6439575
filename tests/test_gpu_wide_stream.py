"""GPU parity of the persistent streaming kernel on codes of 8, 6 and 3 bits at one token: rows of one to eight tiles, prefixes that end
anywhere, row and column segments, with and without zero points, scales of both forms of the bfloat16 unpack, infinite scales behind
the kept columns; against the CPU oracle on sampled rows."""
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
         (2051, 5120, Keep(k_keep=640 * 5, col_seg_stride=8, col_seg_keep=5))]


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
