"""GPU parity of the linears that neither the decode-batch nor the pipelined kernel takes, at the edges of the tiles they run
(csrc/mfma_kernel.h): rows of fewer than eight groups, segments wider than a group or not a power of two, an odd number of kept
columns, a prefix of fewer than eight; against the CPU oracle on all or on sampled rows."""
import numpy as np
import pytest

import workloads as wl
from workloads import Keep
from parity_util import NORM_TOL, NORM_TOL_BF16, TOL, TOL_BF16, linear_err, normwise_err

pytestmark = pytest.mark.gpu


def dev16(torch, a, fmt):
    if fmt == "bf16":
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("M", [2, 9, 16, 17, 32, 33, 48, 64])
@pytest.mark.parametrize("N,K,keep,rows", [
    (131, 896, Keep(n_keep=129, k_keep=893), 16),
    (9700, 896, Keep(n_keep=9665), 64),
    (97, 1280, Keep(k_keep=5 * 216, col_seg_stride=256, col_seg_keep=216), 16),
    (9700, 1280, Keep(k_keep=5 * 216, col_seg_stride=256, col_seg_keep=216), 64),
    (65, 1920, Keep(k_keep=20 * 80, col_seg_stride=96, col_seg_keep=80), 16),
    (9617, 1152, Keep(k_keep=9 * 107, col_seg_stride=128, col_seg_keep=107), 64),
    (33, 1152, Keep(k_keep=5), 16),
])
def test_linear_parity(uref, N, K, keep, rows, M, fmt):
    import torch
    import paper_2512_03383_amd as uq
    rng = wl.rng_for(71, N + M)
    w = wl.gen_linear(rng, N, K, fmt=fmt)
    qw = uq.QuantLinear.from_numpy(w)
    nk, kk = uq.kept_dims(qw, keep)
    x = wl.gen_activations(rng, M, kk, fmt=fmt)
    pick = np.arange(nk) if nk < 1000 else np.unique(np.concatenate([[0, 15, 16, 63, 64, nk - 1], rng.integers(0, nk, rows)]))
    pick = pick.astype(np.int32)
    ref = uref.w4_linear(w["qweight"], w["scales"], w["zeros"], x, keep, fmt=fmt, rows=pick)
    tdt = torch.bfloat16 if fmt == "bf16" else torch.float16
    pad = M % 3
    xb = torch.full((M, kk + pad), float("nan"), dtype=tdt, device="cuda")
    xb[:, :kk] = dev16(torch, x, fmt)
    yb = torch.full((M, nk + pad), -5.0, dtype=tdt, device="cuda")
    uq.uniql_w4_linear(qw, keep, xb[:, :kk], yb[:, :nk])
    torch.cuda.synchronize()
    assert torch.all(yb[:, nk:] == -5.0), "wrote past n_keep"
    y = yb[:, :nk].float().cpu().numpy()[:, pick]
    assert linear_err(y, ref) <= (TOL_BF16 if fmt == "bf16" else TOL)
    if len(pick) >= 64:
        assert normwise_err(y, ref) <= (NORM_TOL_BF16 if fmt == "bf16" else NORM_TOL)
