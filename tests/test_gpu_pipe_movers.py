"""GPU parity of the pipelined kernel's 32 x 32 tiles of 8-bit codes on either side of the row length at which two of four moving waves
stand by (three slabs of 512 columns): prefixes that end anywhere in a block of eight and segments; against the CPU oracle."""
import numpy as np
import pytest

from test_gpu_pipe_tiles import FORMATS, check, env, np16, oracle, weight   # noqa: F401 (env: the fixture)
from workloads import Keep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("M", [17, 40, 64])
@pytest.mark.parametrize("K,keep", [(1024, Keep()), (1536, Keep(k_keep=1529)), (1536, Keep()), (1664, Keep(k_keep=1537)), (1664, Keep(k_keep=1663)), (2048, Keep(k_keep=2045)),
                                    (1536, Keep(k_keep=12 * 102, col_seg_stride=128, col_seg_keep=102)), (1664, Keep(k_keep=26 * 38, col_seg_stride=64, col_seg_keep=38)),
                                    (2176, Keep(k_keep=272 * 6, col_seg_stride=8, col_seg_keep=6))])
def test_rows_around_three_slabs(env, uref, K, keep, M, fmt):   # noqa: F811
    uq, torch = env
    N = 1037
    g = torch.Generator(device="cuda").manual_seed(K + M)
    W = weight(env, g, N, K, 8, fmt)
    kk = uq.kept_dims(W, keep)[1]
    # (decode batches on rows of sixteen groups and more are the ring kernel's)
    assert uq.uniql_w4_linear_kernel(N, K, keep, M, bits=8, bf16=fmt == "bf16", ldx=kk + 1)[:3] == ((1, 32, 16) if M == 17 and K >= 2048 else (2, 32, 32))
    xb = torch.full((M, kk + 1), float("nan"), dtype=W.scales.dtype, device="cuda")
    xb[:, :kk] = torch.randn((M, kk), generator=g, device="cuda").to(W.scales.dtype)
    y = uq.uniql_w4_linear(W, keep, xb[:, :kk])
    torch.cuda.synchronize()
    check(y.float().cpu().numpy(), oracle(uref, W, np.ascontiguousarray(np16(xb[:, :kk], fmt)), keep, fmt, torch.arange(N, device="cuda")), fmt)
