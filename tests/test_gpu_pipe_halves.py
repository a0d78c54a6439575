"""GPU parity of the pipelined kernel's last round of half tiles: grids of a little more than one and two rounds of 256 tiles, whose last
tiles are taken as two halves of the tokens, among them halves without a token; prefixes and segments, against the CPU oracle."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_pipe_tiles import FORMATS, check, env, np16, oracle, weight   # noqa: F401 (env: the fixture)
from workloads import Keep

pytestmark = pytest.mark.gpu


# rows x tokens: 41 x 8 tiles of 128 (328: 72 go out as halves), 66 x 4 (the last token tile has 7 tokens: its second halves are empty), 90 x
# 6 (540: two rounds), 34 x 8 and, in tiles of 96 tokens, 272 and more
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("segments", [False, True])
@pytest.mark.parametrize("bits,N,M", [(8, 5201, 997), (4, 5201, 997), (8, 8400, 391), (6, 8400, 391), (8, 11500, 700), (3, 11500, 700), (4, 4300, 1000), (6, 12185, 333)])
def test_last_round_of_halves(env, uref, bits, N, M, segments, fmt):   # noqa: F811
    uq, torch = env
    K = 1152
    kk = K // 128 * 102 if segments else K - 13
    keep = Keep(n_keep=N - 3, col_seg_stride=128, col_seg_keep=102) if segments else Keep(n_keep=N - 3, k_keep=kk)
    g = torch.Generator(device="cuda").manual_seed(N + M)
    W = weight(env, g, N, K, bits, fmt, zeros=M % 2 == 0)
    x = torch.randn((M, kk), generator=g, device="cuda").to(W.scales.dtype)
    yb = torch.full((M + 2, N), -5.0, dtype=x.dtype, device="cuda")
    uq.uniql_w4_linear(W, keep, x, yb[1:M + 1, :N - 3])
    torch.cuda.synchronize()
    assert torch.all(yb[0] == -5.0) and torch.all(yb[-1] == -5.0) and torch.all(yb[:, N - 3:] == -5.0), "wrote beside the output"
    y = yb[1:M + 1, :N - 3].float().cpu().numpy()
    assert np.isfinite(y).all()
    rng = wl.rng_for(75, N + bits)
    rows = np.unique(np.concatenate([np.arange(0, N - 3, 128), [127, N - 4], rng.integers(0, N - 3, 40)])).astype(np.int64)
    toks = np.unique(np.concatenate([np.arange(0, M, 48), np.arange(63, M, 64), [M - 1], rng.integers(0, M, 8)]))
    cols = Keep(k_keep=kk, col_seg_stride=128, col_seg_keep=102) if segments else Keep(k_keep=kk)
    ref = oracle(uref, W, np.ascontiguousarray(np16(x, fmt)[toks]), cols, fmt, torch.from_numpy(rows).cuda())
    check(y[np.ix_(toks, rows)], ref, fmt)
    # the same bits as in tiles that are taken whole: a few rows by themselves are another grid
    few = uq.QuantLinear(W.qweight[:300].contiguous(), W.scales[:300].contiguous(), W.zeros[:300].contiguous() if W.zeros is not None else None, bits=bits)
    alone = uq.uniql_w4_linear(few, Keep(k_keep=kk, col_seg_stride=128, col_seg_keep=102) if segments else Keep(k_keep=kk), x)
    assert uq.uniql_w4_linear_kernel(300, K, cols, M, bits=bits, bf16=fmt == "bf16", ldx=kk)[0] == 2
    if uq.uniql_w4_linear_kernel(N, K, keep, M, bits=bits, bf16=fmt == "bf16", ldx=kk)[0] == 2:
        assert torch.equal(alone, yb[1:M + 1, :300])
