"""GPU parity of one token on codes of 8 and 6 bits where a row's kept columns end in the lower half of a lane's 32: what is stored for
the upper half does not count, also where its weights lie beyond the largest 16-bit number (and zero times them would be no
number); against the CPU oracle, every row."""
import numpy as np
import pytest

import workloads as wl
from parity_util import NORM_TOL, NORM_TOL_BF16, TOL, TOL_BF16, linear_err, normwise_err
from workloads import Keep

pytestmark = pytest.mark.gpu


def packed(codes, bits):
    """codes [N][K] as the rows' bit streams."""
    b = (codes[:, :, None] >> np.arange(bits)) & 1
    return np.packbits(b.astype(np.uint8).reshape(codes.shape[0], -1), axis=1, bitorder="little").view(np.uint32)


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("bits", [8, 6])
@pytest.mark.parametrize("N,K,kk", [(2563, 4096, 31 * 128 + 16), (2051, 6144, 5 * 1024 + 5), (517, 10240, 78 * 128 + 112), (2561, 4096, 30 * 128 + 81)])
def test_columns_behind_the_last_kept_ones(uref, N, K, kk, bits, fmt):
    import torch
    import paper_2512_03383_amd as uq
    keep, rng, mid = Keep(k_keep=kk), wl.rng_for(76, N + bits), 1 << (bits - 1)
    w = wl.gen_linear8(rng, N, K, fmt=fmt) if bits == 8 else wl.gen_linear_bits(rng, N, K, bits, fmt=fmt)
    codes = rng.integers(0, 2 * mid, (N, K))
    g = kk // 128                                   # the group in which the kept columns end
    near = mid // 8                                 # kept weights of the group are finite: near steps of its scale
    codes[:, g * 128:kk] = rng.integers(mid - near, mid + near, (N, kk - g * 128))
    end = (kk + 15) // 16 * 16
    codes[:, kk:end] = mid
    codes[:, end:] = rng.integers(0, 2, (N, K - end)) * (2 * mid - 1)
    w["qweight"], w["zeros"][:, g] = packed(codes, bits), mid
    # mid - 1 steps overflow, near steps do not
    top = 65504.0 if fmt == "f16" else 2.0 ** 127
    s = np.float32(top / near / 2.1)
    w["scales"].view(np.uint16)[::2, g] = np.float16(s).view(np.uint16) if fmt == "f16" else s.view(np.uint32) >> 16
    x = wl.gen_activations(rng, 1, kk, fmt=fmt)
    xd = torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda().view(torch.bfloat16 if fmt == "bf16" else torch.float16) * 2.0 ** -7
    xn = xd.view(torch.int16).cpu().numpy().view(np.uint16 if fmt == "bf16" else np.float16)
    y = uq.uniql_w4_linear(uq.QuantLinear.from_numpy(w, bits=bits), keep, xd)
    torch.cuda.synchronize()
    ref = uref.wq_linear(bits, w["qweight"], w["scales"], w["zeros"], xn, keep, fmt=fmt)
    assert np.all(np.isfinite(ref)) and np.abs(ref).max() < top
    got = y.double().cpu().numpy()
    for rows in (slice(0, None, 2), slice(1, None, 2)):
        assert linear_err(got[:, rows], ref[:, rows]) <= (TOL_BF16 if fmt == "bf16" else TOL)
        assert normwise_err(got[:, rows], ref[:, rows]) <= (NORM_TOL_BF16 if fmt == "bf16" else NORM_TOL)
