"""GPU parity of the pipelined kernel's 128-token tiles on column segments: whole and partial last blocks of eight, one to sixteen
segments a group, ragged rows and tokens, against the CPU oracle on sampled rows and tokens."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_pipe_tiles import check, env, np16, oracle, weight   # noqa: F401 (env: the fixture)
from workloads import Keep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("bits,stride,keep", [(4, 128, 108), (4, 128, 96), (4, 64, 54), (4, 16, 10), (8, 128, 102), (8, 8, 2), (6, 64, 38), (3, 32, 26)])
def test_128_tokens_of_segments(env, uref, bits, stride, keep, fmt):   # noqa: F811
    uq, torch = env
    N, K, M = 4083, 1152, 1000
    k = Keep(k_keep=K // stride * keep, col_seg_stride=stride, col_seg_keep=keep)
    kk = K // stride * keep
    assert uq.uniql_w4_linear_kernel(N, K, k, M, bits=bits, bf16=fmt == "bf16", ldx=kk + 3)[:2] == (2, 128)
    g = torch.Generator(device="cuda").manual_seed(stride + keep)
    W = weight(env, g, N, K, bits, fmt)
    xb = torch.full((M, kk + 3), float("nan"), dtype=W.scales.dtype, device="cuda")
    xb[:, :kk] = torch.randn((M, kk), generator=g, device="cuda").to(W.scales.dtype)
    y = uq.uniql_w4_linear(W, k, xb[:, :kk])
    torch.cuda.synchronize()
    assert torch.all(torch.isfinite(y))
    rng = wl.rng_for(74, stride + bits)
    rows = np.unique(np.concatenate([[0, 127, 128, 3967, 3968, N - 1], rng.integers(0, N, 60)])).astype(np.int64)
    toks = np.unique(np.concatenate([[0, 127, 128, 895, 896, M - 1], rng.integers(0, M, 14)]))
    ref = oracle(uref, W, np.ascontiguousarray(np16(xb[:, :kk], fmt)[toks]), k, fmt, torch.from_numpy(rows).cuda())
    check(y.float().cpu().numpy()[np.ix_(toks, rows)], ref, fmt)
