"""GPU parity of the pipelined kernel's last round of half tiles: grids of a little more than one and two rounds of 256 tiles, whose last
tiles are taken as two halves of the tokens, among them halves without a token; prefixes and segments, against the CPU oracle."""
import numpy as np
import pytest

import pipe_shapes as ps
import workloads as wl
from test_gpu_pipe_tiles import FORMATS, check, env, np16, oracle, weight   # noqa: F401 (env: the fixture)
from workloads import Keep

pytestmark = pytest.mark.gpu


# grids around the line: 4300 x 1000 and 12185 x 333 have halves of 96-token tiles, the others none (451 and 720 tiles of 96 tokens, 64-token tiles); more with halves
# below
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


def call(env, K, N, M, W, keep, x):   # noqa: F811
    uq, torch = env
    yb = torch.full((M + 2, N), -5.0, dtype=x.dtype, device="cuda")
    uq.uniql_w4_linear(W, keep, x, yb[1:M + 1, :N - 3])
    torch.cuda.synchronize()
    assert torch.all(yb[0] == -5.0) and torch.all(yb[-1] == -5.0) and torch.all(yb[:, N - 3:] == -5.0), "wrote beside the output"
    return yb[1:M + 1, :N - 3]


# grids that have halves, of 128-token tiles too
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("bits,K,N,M,segments,tokens", ps.HALVES)
def test_halves(env, uref, bits, K, N, M, segments, tokens, fmt):   # noqa: F811
    uq, torch = env
    keep = Keep(**ps.halves_rule(K, N, segments))
    g = torch.Generator(device="cuda").manual_seed(N + M)
    W = weight(env, g, N, K, bits, fmt, zeros=bits % 4 == 0)
    x = torch.randn((M, keep.k_keep), generator=g, device="cuda").to(W.scales.dtype)
    kernel, *tile, _ = uq.uniql_w4_linear_kernel(N, K, keep, M, bits=bits, bf16=fmt == "bf16", ldx=keep.k_keep)
    halves, tiles = ps.half_tiles(N - 3, M, tile, torch.cuda.get_device_properties(0).multi_processor_count)
    assert kernel == 2 and tile[0] == tokens and halves > 0
    y = call(env, K, N, M, W, keep, x)
    # rows and tokens at both ends of whole and of half tiles, in the last row tiles above all (the walk ends there)
    rng = wl.rng_for(81, N + bits)
    rows = np.unique(np.concatenate([np.arange(0, N - 3, 640), np.arange(N - 3 - 2 * tile[1], N - 3, 17), [127, N - 4], rng.integers(0, N - 3, 20)])).astype(np.int64)
    toks = np.unique(np.concatenate([np.arange(0, M, tokens // 2), np.arange(tokens // 2 - 1, M, tokens // 2), [M - 1], rng.integers(0, M, 8)]))
    cols = Keep(k_keep=keep.k_keep, col_seg_stride=keep.col_seg_stride, col_seg_keep=keep.col_seg_keep)
    ref = oracle(uref, W, np.ascontiguousarray(np16(x, fmt)[toks]), cols, fmt, torch.from_numpy(rows).cuda())
    check(y.float().cpu().numpy()[np.ix_(toks, rows)], ref, fmt)
    # the same bits for rows in tiles of other grids, none of them halves: the first and the last ones by themselves
    for first in (0, N - 3 - 300):
        part = [None if t is None else t[first:first + 300].contiguous() for t in (W.qweight, W.scales, W.zeros)]
        kernel, *tile, _ = uq.uniql_w4_linear_kernel(300, K, cols, M, bits=bits, bf16=fmt == "bf16", ldx=keep.k_keep)
        assert kernel == 2 and ps.half_tiles(300, M, tile)[0] == 0
        assert torch.equal(uq.uniql_w4_linear(uq.QuantLinear(*part, bits=bits), cols, x), y[:, first:first + 300])
