"""GPU parity of every tile that the pipelined kernel (csrc/pipe_kernel.h) is built with: each code width, format and kind of column
rule, on ragged rows, columns and tokens (tests/pipe_shapes.py; tests/test_linear_routes.py checks on the host that the sizes
take every tile), against the CPU oracle on sampled rows and tokens; column segments of every stride; tokens next to infinities
and NaN."""
import numpy as np
import pytest

import pipe_shapes as ps
import workloads as wl
from parity_util import NORM_TOL, NORM_TOL_BF16, TOL, TOL_BF16, linear_err, normwise_err
from workloads import Keep

pytestmark = pytest.mark.gpu
FORMATS = ["f16", "bf16"]


@pytest.fixture(scope="module")
def env(uref):
    import torch
    import paper_2512_03383_amd as uq
    uq.lib()
    uref.set_threads(min(16, uref.max_threads()))
    return uq, torch


def np16(t, fmt):
    import torch
    a = t.contiguous().view(torch.int16).cpu().numpy()
    return a.view(np.uint16) if fmt == "bf16" else a.view(np.float16)


def weight(env, g, N, K, bits, fmt, zeros=True):
    """Random codes, scales and zero points with the distributions of workloads, made on the device."""
    uq, torch = env
    f = 16.0 / (1 << bits)
    q = torch.randint(-2 ** 31, 2 ** 31, (N, K * bits // 32), generator=g, device="cuda", dtype=torch.int32)
    s = torch.empty((N, K // 128), device="cuda").uniform_(0.005 * f, 0.02 * f, generator=g)
    z = torch.randint(0, 1 << bits, (N, K // 128), generator=g, device="cuda", dtype=torch.uint8) if zeros else None
    return uq.QuantLinear(q, s.to(torch.bfloat16 if fmt == "bf16" else torch.float16), z, bits=bits)


def oracle(uref, W, x, keep_cols, fmt, rows):
    """y of the stored rows `rows` (a row prefix: the compact ones too) from those rows alone."""
    q = W.qweight[rows].cpu().numpy().view(np.uint32)
    s = np16(W.scales[rows], fmt)
    z = W.zeros[rows].cpu().numpy() if W.zeros is not None else None
    if W.bits == 4:
        return uref.w4_linear(q, s, z, x, keep_cols, fmt=fmt)
    return uref.wq_linear(W.bits, q, s, z, x, keep_cols, fmt=fmt)


def check(y, ref, fmt):
    assert linear_err(y, ref) <= (TOL_BF16 if fmt == "bf16" else TOL)
    if ref.shape[1] >= 64:
        assert normwise_err(y, ref) <= (NORM_TOL_BF16 if fmt == "bf16" else NORM_TOL)


@pytest.mark.parametrize("segments", [False, True])
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("bits", [4, 8, 6, 3])
def test_every_tile(env, uref, bits, fmt, segments):
    uq, torch = env
    seen = set()
    for i, (N, K, M) in enumerate(ps.SIZES):
        keep, kk = ps.keep_rule(N, K, segments), ps.kept_columns(K, segments)
        pad = i % 3
        choice = uq.uniql_w4_linear_kernel(N, K, keep, M, bits=bits, bf16=fmt == "bf16", ldx=kk + pad)
        if choice[0] != 2 or choice[1:] in seen:
            continue
        seen.add(choice[1:])
        _, bm, bn, _ = choice
        rng = wl.rng_for(73, N + M + bits)
        g = torch.Generator(device="cuda").manual_seed(N + M)
        W = weight(env, g, N, K, bits, fmt, zeros=i % 2 == 0)
        nk = N - 3
        rows = np.unique(np.concatenate([[0, 15, 16, bn - 1, bn, nk - nk % bn - 1, nk - nk % bn, nk - 2, nk - 1],
                                         rng.integers(0, nk, 70)]).clip(0, nk - 1)).astype(np.int64)
        toks = np.unique(np.concatenate([[0, 15, 16, bm - 1, bm, M - M % bm, M - 1], rng.integers(0, M, 20)]).clip(0, M - 1))
        dt = W.scales.dtype
        xb = torch.full((M, kk + pad), float("nan"), dtype=dt, device="cuda")
        xb[:, :kk] = torch.randn((M, kk), generator=g, device="cuda").to(dt)
        yb = torch.full((M, nk + pad), -5.0, dtype=dt, device="cuda")
        uq.uniql_w4_linear(W, keep, xb[:, :kk], yb[:, :nk])
        torch.cuda.synchronize()
        assert torch.all(yb[:, nk:] == -5.0), "wrote past n_keep"
        assert torch.all(torch.isfinite(yb)), (N, M, choice)
        cols = Keep(k_keep=K // 128 * 102, col_seg_stride=128, col_seg_keep=102) if segments else Keep(k_keep=kk)
        ref = oracle(uref, W, np.ascontiguousarray(np16(xb[:, :kk], fmt)[toks]), cols, fmt, torch.from_numpy(rows).cuda())
        check(yb[:, :nk].float().cpu().numpy()[np.ix_(toks, rows)], ref, fmt)
    assert seen == ps.tiles(bits, segments)


# strides of 8 to 128 columns, segments that keep two columns up to all but two, even numbers (4 bits: eight columns at least, others
# are another kernel's)
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("bits,stride,keep", [
    (bits, stride, keep) for bits in (4, 8, 6, 3)
    for stride, keep in ((8, 2), (8, 6), (16, 4), (16, 10), (16, 14), (32, 6), (32, 8), (32, 26), (64, 2), (64, 38), (128, 4), (128, 94), (128, 126))
    if bits != 4 or keep >= 8])
def test_segments_of_every_stride(env, uref, bits, stride, keep, fmt):
    uq, torch = env
    for N, K, M in ((600, 1280, 40), (260, 1152, 130)):
        k = Keep(k_keep=K // stride * keep, col_seg_stride=stride, col_seg_keep=keep)
        kk = K // stride * keep
        assert uq.uniql_w4_linear_kernel(N, K, k, M, bits=bits, bf16=fmt == "bf16", ldx=kk)[0] == 2
        g = torch.Generator(device="cuda").manual_seed(stride + keep)
        W = weight(env, g, N, K, bits, fmt)
        x = torch.randn((M, kk), generator=g, device="cuda").to(W.scales.dtype)
        y = uq.uniql_w4_linear(W, k, x)
        torch.cuda.synchronize()
        check(y.float().cpu().numpy(), oracle(uref, W, np16(x, fmt), k, fmt, torch.arange(N, device="cuda")), fmt)


# what stands in one token does not reach its neighbours: rows of infinities and NaN among finite ones, prefixes that end anywhere in
# a block of eight and segments, whose last block is read with the next token's first columns behind it
@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("bits", [4, 8, 6, 3])
@pytest.mark.parametrize("K,keep", [(1152, Keep(k_keep=1145)), (1152, Keep(k_keep=1150)), (1152, Keep()), (1280, Keep(k_keep=1029)),
                                    (1152, Keep(k_keep=9 * 102, col_seg_stride=128, col_seg_keep=102)),
                                    (1280, Keep(k_keep=40 * 26, col_seg_stride=32, col_seg_keep=26))])
@pytest.mark.parametrize("N,M", [(600, 40), (6500, 50), (260, 130)])
def test_tokens_next_to_infinities(env, uref, N, M, K, keep, bits, fmt):
    uq, torch = env
    g = torch.Generator(device="cuda").manual_seed(K + M)
    W = weight(env, g, N, K, bits, fmt)
    kk = uq.kept_dims(W, keep)[1]
    assert uq.uniql_w4_linear_kernel(N, K, keep, M, bits=bits, bf16=fmt == "bf16", ldx=kk)[0] == 2
    x = torch.randn((M, kk), generator=g, device="cuda").to(W.scales.dtype)
    clean = uq.uniql_w4_linear(W, keep, x)
    bad = torch.arange(M, device="cuda") % 3 == 1
    x2 = x.clone()
    x2[bad] = torch.where(torch.rand((int(bad.sum()), kk), generator=g, device="cuda") < 0.5, float("inf"), float("nan")).to(x.dtype)
    y = uq.uniql_w4_linear(W, keep, x2)
    torch.cuda.synchronize()
    assert torch.equal(y[~bad], clean[~bad]) and torch.all(torch.isfinite(clean))
